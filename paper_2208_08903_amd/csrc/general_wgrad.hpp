// Weight gradients of the general kernels in FP32,
//   dW[co][ci][t] = sum over (sample, site) of g[n][co] u[n + delta_t][ci],  db[co] = sum g[n][co],
// from a group of layers' activations and gradients in quad planes (see net_engine.hpp).
//
// A workgroup takes 16 rows (co) and up to 16 channels ci of one convolution of one layer,
// sample after sample.  A slab of the leading axis at a time lies in LDS: g as it is, u with
// its periodic halo, so that the neighbour at a tap is a fixed distance from a site's place
// and a column, a (tap, channel) pair, is a fixed offset of its lane.  50 samples of 12^3,
// hidden 16, 12 layers: 1254 us with FP64 MFMAs on operands addressed and read from the L2
// one by one, 591 us so, of which the MFMAs are 210 (two of three convolutions; the last one
// has 2 rows of 16) and most of the rest the second round of 1200 workgroups on 512 places.
//
// The sums, as direct kernels form them:
//   CHAIN  (Seq) a sample's sites one after the other by FP32 fused multiply-adds, which is
//          v_mfma_f32_16x16x4_f32 with four sites as its k; samples in FP64
//   else   products rounded to FP32, added in FP64: v_mfma_f64_16x16x4_f64 adds the exact
//          products, and the FP32 units the roundings' errors g u - fl(g u), exact in FP32 and
//          2^-24 of them, which are taken off at the end (64 samples of 8 x 8, hidden
//          [16, 16, 16], 16 layers: 154 us with the products converted and added one by one,
//          85 so; 55 with exact products, whose sums round to other gradients, however)
#pragma once

#include "general_common.hpp"

namespace lfs {
namespace {

constexpr int kWsCols = 3;  // column tiles of a wave
struct WsConv {
  int rows, rt;           // output channels, in tiles of 16
  int cw, ncb;            // channels of a column block (1: the field), column blocks
  Magic dcw;
  int tiles, groups;      // column tiles of a block, in groups of one workgroup's
  int gplane, gplanes, uplane, uplanes;  // planes of g and u in the store
  int slices;             // of the leading axis per slab
  int us, gs;             // plane strides in LDS, floats
  int job0;
};
struct WsArgs {
  WsConv c[kMaxConv];
  int jobs, waves;        // workgroups per (layer, chunk); waves with columns, CHAIN: one more for db
  int planes;             // planes of a sample's block of the store
  int l0, layers, B, chunks, per;  // per: samples of a chunk
  int parts;              // or, above 1, chunks of one part of a sample's leading axis each
  Magic dLp;              // L + 2 (K / 2)
  int lds;
};

template <int DIM, bool CHAIN>
__global__ void __launch_bounds__(1024) kg_wgrad_slab(NetDev d, WsArgs A, const float* __restrict__ store,
                                                      const float* __restrict__ saved, double* __restrict__ partial) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  constexpr int CT = kWsCols;
  extern __shared__ __align__(16) unsigned char smem[];
  const Lat& lat = d.lat;
  const int L = lat.L, V = lat.V, lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4, w = fused::wave_id();
  const int ll = blockIdx.x, job = A.jobs - 1 - (int)blockIdx.z, layer = A.l0 + ll;  // the first convolution's come last
  int i = 0;
  while (i + 1 < d.n_conv && job >= A.c[i + 1].job0) ++i;
  const WsConv C = A.c[i];
  int r = job - C.job0;
  const int tg = r % C.groups;
  r /= C.groups;
  const int cb = r % C.ncb, rt = r / C.ncb;
  const bool field = i == 0;
  const int fpar = (layer + d.parity0) & 1, h = d.K >> 1, Lp = L + 2 * h;
  const int area = DIM == 2 ? L : L * L, parea = DIM == 2 ? Lp : Lp * Lp;  // a slice, plain and with halo
  const int gp = min(4, C.gplanes - 4 * rt), up = field ? 1 : min(C.cw >> 2, C.uplanes - cb * (C.cw >> 2));
  const int smax = C.slices * area, s4 = (smax + 3) & ~3;
  uint32_t* place = reinterpret_cast<uint32_t*>(smem);  // of a slab's sites among u's
  float* gl = reinterpret_cast<float*>(smem) + s4;
  float* ul = gl + gp * C.gs;
  for (int n = threadIdx.x; n < s4; n += blockDim.x) {
    const int nn = min(n, smax - 1);
    int row = fdiv(nn, lat.dL), q = nn - row * L;
    if constexpr (DIM == 3) {
      const int z = fdiv(row, lat.dL);
      row += 2 * h * z;  // z Lp + y
    }
    place[n] = (uint32_t)(row * Lp + q) * (field ? 1 : 4);
  }
  // the wave's columns: offsets of u from a site's place; rows of g
  int coff[CT];
  const int t0 = (tg * A.waves + w) * CT;
#pragma unroll
  for (int q = 0; q < CT; ++q) {
    const int f = min((t0 + q) * 16 + m, d.T * C.cw - 1), tap = fdiv(f, C.dcw), ch = f - tap * C.cw;
    int o = 0, t = tap, pitch = 1;
#pragma unroll
    for (int mu = 0; mu < DIM; ++mu) {  // the fastest axis is the last digit
      const int k = fdiv(t, d.dK);
      o += (t - k * d.K) * pitch;
      pitch *= Lp;
      t = k;
    }
    coff[q] = field ? o : min(ch >> 2, up - 1) * C.us + 4 * o + (ch & 3);
  }
  const int groff = min(m >> 2, gp - 1) * C.gs + (m & 3);
  const bool cols = w < A.waves && t0 < C.tiles, bias = w == (CHAIN ? A.waves : 0) && cb == 0 && tg == 0;
  f32x4 acc[CHAIN ? CT : 1];
  f64x4 sum[CT];  // D of an MFMA, FP64: row 4 k + kk; FP32: 4 kk + k
  float err[CHAIN ? 1 : CT][16], b32 = 0.f;
  double bsum = 0.0;
#pragma unroll
  for (int q = 0; q < CT; ++q) {
    sum[q] = f64x4{0.0, 0.0, 0.0, 0.0};
    if constexpr (!CHAIN)
#pragma unroll
      for (int k = 0; k < 16; ++k) err[q][k] = 0.f;
  }
  const int b0 = blockIdx.y / A.parts * A.per, b1 = min(b0 + A.per, A.B), part = blockIdx.y % A.parts;
  const int zlo = L * part / A.parts, zhi = L * (part + 1) / A.parts;
  for (int b = b0; b < b1; ++b) {
    const float* st = store + ((size_t)ll * A.B + b) * A.planes * V * 4;
    const float* sx = saved + ((size_t)layer * A.B + b) * V;
    if constexpr (CHAIN) {
#pragma unroll
      for (int q = 0; q < CT; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      b32 = 0.f;
    }
    for (int z0 = zlo; z0 < zhi; z0 += C.slices) {
      const int ns = min(C.slices, zhi - z0) * area, n4 = (ns + 3) & ~3;
      __syncthreads();  // the last slab's readers
      for (int n = threadIdx.x; n < n4; n += blockDim.x)
        for (int p = 0; p < gp; ++p) {
          f32x4 v{0.f, 0.f, 0.f, 0.f};
          if (n < ns)
            v = *reinterpret_cast<const f32x4*>(st + ((size_t)(C.gplane + 4 * rt + p) * V + z0 * area + n) * 4);
          *reinterpret_cast<f32x4*>(gl + p * C.gs + 4 * n) = v;
        }
      const int np = (min(C.slices, zhi - z0) + 2 * h) * parea;
      for (int e = threadIdx.x; e < np; e += blockDim.x) {
        // padded coordinates to a site, fastest axis last
        int c[DIM], q = e;
#pragma unroll
        for (int mu = DIM - 1; mu > 0; --mu) {
          const int k = fdiv(q, A.dLp);
          c[mu] = q - k * Lp;
          q = k;
        }
        c[0] = q + z0;
        int n = 0, par = 0;
#pragma unroll
        for (int mu = 0; mu < DIM; ++mu) {
          int x = c[mu] - h;
          while (x < 0) x += L;
          while (x >= L) x -= L;
          n = n * L + x;
          par ^= x;
        }
        if (field) {
          ul[e] = masked(sx[n], ((par & 1) ^ fpar) - 1);
        } else {
          for (int p = 0; p < up; ++p)
            *reinterpret_cast<f32x4*>(ul + p * C.us + 4 * e) = *reinterpret_cast<const f32x4*>(
                st + ((size_t)(C.uplane + cb * (C.cw >> 2) + p) * V + n) * 4);
        }
      }
      __syncthreads();
      if (cols) {
        const int steps = n4 >> 2, last = steps - 1;
        struct Op {
          float a, v[CT];
        };
        // step k's operands, the sites' places looked up a step earlier; u is read as zero
        // past the slab, as g is (it need not be finite there)
        auto load = [&](int k, uint32_t at) {
          const int n = 4 * k + kk, in = (n - ns) >> 31;
          Op o;
          o.a = gl[groff + 4 * n];
#pragma unroll
          for (int q = 0; q < CT; ++q) o.v[q] = masked(ul[at + coff[q]], in);
          return o;
        };
        // operands two steps ahead: three MFMAs are shorter than the LDS's latency
        Op o = load(0, place[kk]), o1 = load(min(1, last), place[4 * min(1, last) + kk]);
        uint32_t at = place[4 * min(2, last) + kk];
        for (int k = 0; k < steps; ++k) {
          const Op o2 = load(min(k + 2, last), at);
          at = place[4 * min(k + 3, last) + kk];
          if constexpr (CHAIN) {
#pragma unroll
            for (int q = 0; q < CT; ++q) acc[q] = fused::mfma(o.a, o.v[q], acc[q]);
          } else {
#pragma unroll
            for (int q = 0; q < CT; ++q)
              sum[q] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)o.a, (double)o.v[q], sum[q], 0, 0, 0);
            bsum += (double)o.a;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
              if (p < gp) {
                const f32x4 g = *reinterpret_cast<const f32x4*>(gl + p * C.gs + 16 * k + 4 * kk);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                  for (int q = 0; q < CT; ++q)
                    err[q][4 * p + e] += __builtin_fmaf(g[e], o.v[q], -__fmul_rn(g[e], o.v[q]));
              }
            }
          }
          o = o1;
          o1 = o2;
        }
      }
      if constexpr (CHAIN)
        if (bias && lane < 16)
#pragma unroll 8
          for (int n = 0; n < n4; ++n) b32 += gl[groff + 4 * n];
    }
    if constexpr (CHAIN) {
#pragma unroll
      for (int q = 0; q < CT; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) sum[q][k] += (double)acc[q][k];
      bsum += (double)b32;
    }
  }
  double* out = partial + ((size_t)blockIdx.y * A.layers + ll) * d.P_layer;
  const bool gseq = CHAIN && i + 1 < d.n_conv, useq = CHAIN && i > 0;
  if (cols) {
#pragma unroll
    for (int q = 0; q < CT; ++q) {
      const int f = (t0 + q) * 16 + m, tap = fdiv(f, C.dcw), ch = f - tap * C.cw;
      const int ci = field ? 0 : chan_of(useq, d.cin[i], cb * (C.cw >> 2) + (ch >> 2), ch & 3);
      const bool ok = tap < d.T && ci < d.cin[i] && (field || (ch >> 2) < up);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        double v = sum[q][k];
        if constexpr (!CHAIN) {
          double e = 0.0;
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            double y = (double)err[q][4 * k + x];
            y += __shfl_xor(y, 16);
            y += __shfl_xor(y, 32);
            e = kk == x ? y : e;
          }
          if (__builtin_isfinite(e)) v -= e;  // (not where a product is infinite)
        }
        const int row = CHAIN ? 4 * kk + k : 4 * k + kk, pl = row >> 2;
        const int co = chan_of(gseq, d.cout[i], 4 * rt + pl, row & 3);
        if (ok && pl < gp && co < d.cout[i]) out[d.offW[i] + (co * d.cin[i] + ci) * d.T + tap] = v;
      }
    }
  }
  if constexpr (!CHAIN) {
    bsum += __shfl_xor(bsum, 16);
    bsum += __shfl_xor(bsum, 32);
  }
  if (bias && lane < 16 && (m >> 2) < gp) {
    const int co = chan_of(gseq, d.cout[i], 4 * rt + (m >> 2), m & 3);
    if (co < d.cout[i]) out[d.offb[i] + co] = bsum;
  }
}

// The slab kernel's plan for `layers` layers of B samples; lds = 0 where a slab of one slice
// and four channels does not fit the LDS.
struct WsPlan {
  WsArgs a;
  size_t partial_bytes;
};
WsPlan wgrad_slab_plan(const NetDev& d, int B, int layers, int planes) {
  WsPlan p{};
  WsArgs& a = p.a;
  const int n = d.n_conv, L = d.lat.L, h = d.K / 2, Lp = L + 2 * h;
  const int64_t area = d.dim == 2 ? L : (int64_t)L * L, parea = d.dim == 2 ? Lp : (int64_t)Lp * Lp;
  auto stride = [](int64_t floats) { return (floats + 47) / 64 * 64 + 16; };  // 16 mod 64: planes in other banks
  auto bytes = [&](const WsConv& c, int i, int64_t s) {
    const int64_t up = i == 0 ? 1 : c.cw / 4, us = i == 0 ? stride((s + 2 * h) * parea) : stride(4 * (s + 2 * h) * parea);
    return 4 * ((s * area + 3) / 4 * 4 + std::min(4, c.gplanes) * stride(4 * (s * area + 3)) + up * us);
  };
  int most = 0;
  for (int i = 0; i < n; ++i) {
    WsConv& c = a.c[i];
    c.rows = d.cout[i];
    c.rt = cdiv(c.rows, 16);
    c.gplane = i + 1 < n ? d.hplanes + d.hplane[i] : 2 * d.hplanes;
    c.gplanes = cdiv(d.cout[i], 4);
    c.uplane = i > 0 ? d.hplane[i - 1] : 0;
    c.uplanes = cdiv(d.cin[i], 4);
    c.cw = i == 0 ? 1 : 4 * std::min(4, c.uplanes);
    // fewer channels where even a slab of one slice does not fit
    while (i > 0 && c.cw > 4 && bytes(c, i, 1) > kLdsMax) c.cw -= 4;
    if (bytes(c, i, 1) > kLdsMax) return WsPlan{};
    c.dcw = magic(c.cw);
    c.ncb = i == 0 ? 1 : cdiv(c.uplanes * 4, c.cw);
    c.tiles = cdiv(d.T * c.cw, 16);
    most = std::max(most, c.tiles);
  }
  a.waves = std::min(15, cdiv(most, kWsCols));
  // the thickest slab, or one slice, that leaves room for two workgroups per CU, for more where
  // they have few waves: 16 waves a CU, or eight workgroups
  const int64_t room = d.mode == kSeq ? 78 * 1024 : std::clamp(156 * 1024 * a.waves / 16, 19 * 1024, 78 * 1024);
  for (int i = 0; i < n; ++i) {
    WsConv& c = a.c[i];
    int s = 1;
    while (s < L && bytes(c, i, s + 1) <= room) ++s;
    s = cdiv(L, cdiv(L, s));
    c.slices = s;
    c.gs = (int)stride(4 * (s * area + 3));
    c.us = (int)(i == 0 ? stride((s + 2 * h) * parea) : stride(4 * (s + 2 * h) * parea));
    a.lds = std::max(a.lds, (int)bytes(c, i, s));
  }
  int job = 0;
  for (int i = 0; i < n; ++i) {
    WsConv& c = a.c[i];
    c.groups = cdiv(c.tiles, a.waves * kWsCols);
    c.job0 = job;
    job += c.rt * c.ncb * c.groups;
  }
  a.dLp = magic(Lp);
  a.jobs = job;
  a.layers = layers;
  a.planes = planes;
  a.B = B;
  // about 2048 workgroups of whole samples.  Where these make fewer than 2048 waves, each sample
  // is cut along its leading axis, in parts of 64 sites or more and no thinner than half their
  // halo (not in Seq, whose sums over a sample are FP32).  Four samples of 256 x 256, hidden [1], kernel 1, 2
  // layers: 5537 us with whole samples, 87 with parts of them; three of 32^3, hidden [2, 4]: 2790
  // and 207.  (98 of 8 x 8, hidden [16, 12, 4], kernel 7, which fill the chip, cut in two: a
  // training step of 4 layers 454 -> 544 us.)
  const int64_t each = (int64_t)job * layers, want = std::max<int64_t>(1, 2048 / each);
  a.per = cdiv(B, (int)std::min<int64_t>(B, want));
  a.parts = 1;
  if (d.mode != kSeq && each * B * a.waves < 2048)
    a.parts = std::max(1, std::min({L / std::max(1, h), d.lat.V / 64, cdiv((int)(4096 / (each * a.waves)), B)}));
  a.chunks = cdiv(B, a.per) * a.parts;
  p.partial_bytes = sizeof(double) * (size_t)a.chunks * layers * d.P_layer;
  return p;
}

// Weight gradients of layers [l0, l0 + layers) from their store into g_params.
template <int DIM, int MODE>
int32_t run_wgrad(const NetDev& d, int B, int l0, int layers, int planes, const float* store, const float* saved,
                  double* partial, float* g_params, hipStream_t st) {
  const int n = layers * d.P_layer;
  int chunks;
  WsPlan s{};
  if constexpr (MODE != kBf16) s = wgrad_slab_plan(d, B, layers, planes);
  if (s.a.lds && MODE != kBf16) {
    s.a.l0 = l0;
    chunks = s.a.chunks;
    constexpr auto k = kg_wgrad_slab<DIM, MODE == kSeq>;
    if (!set_lds_limit<k>(kLdsMax)) return LFS_EDEVICE;
    hipLaunchKernelGGL(k, dim3((unsigned)layers, (unsigned)chunks, (unsigned)s.a.jobs),
                       dim3(64 * (s.a.waves + (MODE == kSeq))), s.a.lds, st, d, s.a, store, saved, partial);
  } else {
    WgPlan p = wgrad_plan(d, B, layers, planes);
    p.a.l0 = l0;
    chunks = p.a.chunks;
    hipLaunchKernelGGL((kg_wgrad<DIM, MODE == kBf16>), dim3((unsigned)(p.a.jobs * layers), (unsigned)chunks),
                       dim3(256), 0, st, d, p.a, store, saved, partial);
  }
  if (chunks > kRedChunks)
    hipLaunchKernelGGL(kg_reduce<16>, dim3(blocks(n, 64)), dim3(1024), 0, st, d, n, chunks, partial,
                       g_params + (size_t)l0 * d.P_layer);
  else
    hipLaunchKernelGGL(kg_reduce<1>, dim3(blocks(n)), dim3(256), 0, st, d, n, chunks, partial,
                       g_params + (size_t)l0 * d.P_layer);
  return LFS_OK;
}

// Bytes of the partial sums of groups of `group` layers (the last one may be smaller and
// take more chunks).
size_t partial_bytes(const NetDev& d, int B, int group, int planes) {
  auto of = [&](int layers) {
    size_t b = wgrad_plan(d, B, layers, planes).partial_bytes;
    if (d.mode != kBf16) {
      const WsPlan s = wgrad_slab_plan(d, B, layers, planes);
      if (s.a.lds) b = s.partial_bytes;
    }
    return b;
  };
  size_t pb = of(group);
  if (d.N % group) pb = std::max(pb, of(d.N % group));
  return pb;
}

}  // namespace
}  // namespace lfs
