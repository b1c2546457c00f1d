// Kernels and host pieces shared by the general kernels with and without batch norm:
// fragment preparation, one convolution over a workgroup's sample in LDS, the weight
// gradients and their reduction.
#pragma once

#include <algorithm>
#include <type_traits>

#include "net_engine.hpp"

namespace lfs {
namespace {  // each translation unit keeps its own copy of the kernels

using namespace net;

constexpr double kHalfLog2Pi = 0.91893853320467274178;
constexpr size_t kLdsMax = 158 * 1024;

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One thread per (layer, fragment, lane): fragments f0 .. f0 + count - 1 of every layer.
template <int MODE>
__global__ void __launch_bounds__(256) kg_prep(NetDev d, const float* __restrict__ params, int layers, int f0,
                                               int count, u32x4* __restrict__ frags) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)layers * count * 64) return;
  const int lane = (int)(gid & 63);
  const int64_t fl = gid >> 6;
  const int layer = (int)(fl / count), f = f0 + (int)(fl - (int64_t)layer * count);
  const bool tr = f >= d.frags_fwd;
  int i = 0;
  for (; i + 1 < d.n_conv; ++i)
    if (f < (tr ? d.t[i + 1] : d.f[i + 1]).off) break;
  const ConvDir& c = tr ? d.t[i] : d.f[i];
  const int r = f - c.off, ct = r / c.per_ct();
  frags[gid] = frag_entry<MODE>(d, params + (size_t)layer * d.P_layer, i, tr, ct, r - ct * c.per_ct() - 1, lane);
}

// Waves of a resident workgroup at most (of so many, small lattices split the K blocks of a
// unit over them).
constexpr int kResWaves = 8;

// Copies n fragments to LDS without passing through registers: 1 KB per instruction, lane
// i's 16 bytes at the fragment's LDS address + 16 i.  Counts as vector-memory loads.
__device__ __forceinline__ void copy_frags(const u32x4* src, unsigned char* dst, int n) {
  typedef __attribute__((address_space(1))) void* gptr;
  typedef __attribute__((address_space(3))) void* lptr;
  const int lane = threadIdx.x & 63;
  for (int k = fused::wave_id(); k < n; k += blockDim.x >> 6)
    __builtin_amdgcn_global_load_lds((gptr)(src + (size_t)k * 64 + lane), (lptr)(dst + k * 1024), 16, 0, 0);
}
__device__ __forceinline__ void wait_copies() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

// One convolution over (16-site tile, row tile) units: a wave per unit, or, where that leaves
// SIMDs idle, four waves per unit (Bf16: also two, and two waves per SIMD), each on its share
// of the K blocks (Tree: of the eight sums; Seq keeps its order and is not split), joined
// through red.  A Tree unit per SIMD is faster whole: split, the four waves of a SIMD took
// as long over its MFMAs and four times the LDS reads (two floats of each 32 bytes).  reader(tile) gives the operand reader of the lane's
// site, epi(tile, ct, acc) takes a unit's result.  FEW: the workgroup may have fewer waves than
// kResWaves; in Bf16 a wave then makes all shares of its unit, in the same order (compiled
// apart: beside the other path it cost that 4 %).  Ends before any barrier that publishes
// epi's stores.
template <int MODE, bool TR, bool FEW, class Reader, class Epi>
__device__ __forceinline__ void conv_pass(int tiles, const ConvDir& cd, const u32x4* frags, f32x4* red,
                                          Reader&& reader, Epi&& epi) {
  const int w = fused::wave_id(), nw = blockDim.x >> 6, lane = threadIdx.x & 63, j = lane >> 4;
  const int nct = cd.nct, units = tiles * nct;
  const ConvDir c = cd;
  const Weights W{frags, c.per_ct(), lane};
  constexpr bool TREE = MODE == kTree;
  int sh = 0;  // a unit in 2^sh shares
  if constexpr (TREE)
    sh = !FEW && units <= 2 ? 2 : 0;
  else if constexpr (MODE == kBf16)
    while (sh < 2 && (2 * units << sh) <= kResWaves && (2 << sh) <= c.nb) ++sh;
  const int ks = 1 << sh;
  auto bias = [&](int ct) { return __builtin_bit_cast(f32x4, W.at(ct, -1)); };
  if (sh == 0 || FEW) {
    for (int u = w; u < units; u += nw) {
      const int tile = fdiv(u, c.dnct), ct = u - tile * nct;
      const auto rd = reader(tile);
      if constexpr (TREE) {
        epi(tile, ct, TR ? tree<false>(rd, c, W, ct, j, 0) : tree<false>(rd, c, W, ct, j, 0) + bias(ct));
      } else {
        f32x4 acc = chain<MODE, TR>(rd, c, W, ct, j, 0, c.nb >> sh, bias(ct));
        if constexpr (FEW)
          for (int p = 1; p < ks; ++p)
            acc += chain<MODE, TR>(rd, c, W, ct, j, c.nb * p >> sh, c.nb * (p + 1) >> sh, f32x4{0.f, 0.f, 0.f, 0.f});
        epi(tile, ct, acc);
      }
    }
    return;
  }
  const int kp = (w >= units) + (w >= 2 * units) + (w >= 3 * units) + (w >= 4 * units), u = w - kp * units;
  const int tile = fdiv(u, c.dnct), ct = u - tile * nct;
  f32x4 acc{0.f, 0.f, 0.f, 0.f};
  if (kp < ks) {
    const auto rd = reader(tile);
    if constexpr (TREE) {
      acc = tree<true>(rd, c, W, ct, j, kp);
    } else {
      if (kp == 0) acc = bias(ct);
      acc = chain<MODE, TR>(rd, c, W, ct, j, c.nb * kp >> sh, c.nb * (kp + 1) >> sh, acc);
    }
    if (kp > 0) red[((kp - 1) * units + u) * 64 + lane] = acc;
  }
  lds_barrier();
  if (kp == 0) {
    if constexpr (TREE) {
      const f32x4 p1 = red[u * 64 + lane], p2 = red[(units + u) * 64 + lane], p3 = red[(2 * units + u) * 64 + lane];
      acc = (acc + p2) + (p1 + p3);
      if constexpr (!TR) acc += bias(ct);
    } else {
      for (int p = 0; p + 1 < ks; ++p) acc += red[(p * units + u) * 64 + lane];
    }
    epi(tile, ct, acc);
  }
}

// The reader of input planes at `in` (stride ps floats) for site n, neighbour table nbr.
template <bool REV>
__device__ __forceinline__ Planes<REV, true> lds_planes(const NetDev& d, const uint16_t* nbr, int ps, const float* in,
                                                     int n) {
  return Planes<REV, true>{nbr + d.lat.V + n, in, d.lat.V, ps, d.T};
}

// The reader of the masked field xm for site n.
__device__ __forceinline__ Field<true> lds_field(const NetDev& d, const uint16_t* nbr, const float* xm, int n) {
  return Field<true>{nbr + d.lat.V + n, xm, d.lat.V, d.T};
}

// Plane stride in LDS, floats: the site after the last one is kept at zero, and 16 mod 64
// lets the planes of a gather's four lane groups start in different banks.
inline int lds_plane_stride(int V) { return (4 * (V + 1) + 47) / 64 * 64 + 16; }

// Affine backward at an active site from o_0: g_o into (go0, g) and g_x.
__device__ __forceinline__ void affine_bwd(int final_tanh, float o0, float x, float g, float gld, float& go0,
                                           float& gx) {
  const float s = final_tanh ? tanhf(o0) : o0;
  const float es = expf(s);
  const float gs = g * x * es + gld;
  go0 = final_tanh ? gs * (1.f - s * s) : gs;
  gx = g * es;
}

// v(0) + .. + v(n - 1) by one wave, in the order of block_sum over 256 threads that take every
// 256th.
template <class T, class F>
__device__ __forceinline__ T sum_of_256(int n, F&& v) {
  const int lane = threadIdx.x & 63;
  T r = 0;
  for (int w = 0; w < 4 && 64 * w < n; ++w) {
    T acc = 0;
    for (int t = 64 * w + lane; t < n; t += 256) acc += v(t);
    acc = wave_sum(acc);
    r = w == 0 ? acc : r + acc;
  }
  return r;
}

// log r of a sample of V sites from the sum of its squares.
__device__ __forceinline__ double log_prior(int V, double zz) { return -0.5 * zz - (double)V * kHalfLog2Pi; }

// log r(z) per sample and the first field: saved[0], or phi (which may be z).
template <typename R>
__global__ void __launch_bounds__(256) kg_begin(int V, const float* z, float* x, double* __restrict__ logr) {
  __shared__ R sh[16];
  const int b = blockIdx.x;
  R acc = 0;
  for (int n = threadIdx.x; n < V; n += blockDim.x) {
    const float v = z[(size_t)b * V + n];
    if (x != z) x[(size_t)b * V + n] = v;
    acc += (R)v * v;
  }
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) logr[b] = log_prior(V, (double)acc);
}

// ---- weight gradients --------------------------------------------------------------

// (BF16, and lattices of which a slab does not fit the LDS; else general_wgrad.hpp.)
// dW[co][ci][t] = sum over (sample, site) of g[n][co] u[n + delta_t][ci] as GEMMs over the
// sites on v_mfma_f64_16x16x4_f64: products of FP32 values are exact and every sum is
// FP64.  Rows are 16 channels of the operand read in place, columns 16 (tap, channel)
// pairs of the other one, read displaced: u displaced (rows co), or, where that takes
// fewer tiles (the last convolution, whose g has two channels), g displaced the other
// way (rows ci).
struct WgConv {
  int swap;               // 1: rows are ci, columns (tap, co) with g displaced by -delta
  int rows, ncols, cc;    // row channels, T * cc columns, channels per tap
  int rt, groups;         // row tiles, groups of kWgCols column tiles
  int gplane, uplane;     // first planes of g and u in the store (u of the first: the field)
  int gseq, useq;         // their planes hold channels in Seq order
  int job0;               // first job
};
constexpr int kWgCols = 3;   // column tiles of a wave (12 accumulator registers pairs each)
constexpr int kWgUnroll = 4;
struct WgArgs {
  WgConv c[kMaxConv];
  int jobs;               // per layer
  int planes;             // planes of a sample's block of the store
  int l0, layers, B, chunks;
  int64_t per;            // (sample, site) terms per chunk, a multiple of 16
};

template <int DIM, bool BF16>
__global__ void __launch_bounds__(256) kg_wgrad(NetDev d, WgArgs A, const float* __restrict__ store,
                                                const float* __restrict__ saved, double* __restrict__ partial) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  __shared__ double red[4][64][4];
  __shared__ double redb[4][64];
  const Lat& lat = d.lat;
  const int V = lat.V, lane = threadIdx.x & 63, m = lane & 15, kk = lane >> 4, w = fused::wave_id();
  const int ll = blockIdx.x / A.jobs, job = blockIdx.x - ll * A.jobs, layer = A.l0 + ll;
  int i = 0;
  while (i + 1 < d.n_conv && job >= A.c[i + 1].job0) ++i;
  const WgConv& C = A.c[i];
  const int r = job - C.job0, rt = r / C.groups, cg = r - rt * C.groups;
  const int fpar = (layer + d.parity0) & 1, PL = A.planes;
  // the lane's row channel and its (tap, channel) column of every column tile
  const int row = rt * 16 + m;
  const bool rok = row < C.rows;
  const int rch = rok ? row : 0;
  int ent[kWgCols], cch[kWgCols], coff[kWgCols];
  bool cok[kWgCols];
#pragma unroll
  for (int q = 0; q < kWgCols; ++q) {
    const int f = (cg * kWgCols + q) * 16 + m;
    cok[q] = f < C.ncols;
    const int tap = cok[q] ? f / C.cc : 0;
    cch[q] = cok[q] ? f - tap * C.cc : 0;
    ent[q] = tap_entry<DIM>(d, tap, C.swap ? -1 : 1);
  }
  const bool first = i == 0;
  // operand offsets within a sample's store block; the first convolution's u is the field
  int roff;
  {
    int pl, e;
    place_of(C.swap ? C.useq : C.gseq, C.swap ? d.cin[i] : d.cout[i], rch, pl, e);
    roff = ((C.swap ? C.uplane : C.gplane) + pl) * V * 4 + e;
#pragma unroll
    for (int q = 0; q < kWgCols; ++q) {
      place_of(C.swap ? C.gseq : C.useq, C.swap ? d.cout[i] : d.cin[i], cch[q], pl, e);
      coff[q] = ((C.swap ? C.gplane : C.uplane) + pl) * V * 4 + e;
    }
  }
  const bool row_x = first && C.swap, col_x = first && !C.swap;
  const int64_t terms = (int64_t)A.B * V, c0 = (int64_t)blockIdx.y * A.per, c1 = min(c0 + A.per, terms);
  // each wave a quarter of the chunk, in steps of four terms (lane group kk: the kk-th)
  const int64_t quarter = ((c1 - c0 + 15) / 16) * 4;
  const int64_t w0 = min(c0 + w * quarter, c1), w1 = min(w0 + quarter, c1);
  f64x4 acc[kWgCols];
  double bias = 0.0;
#pragma unroll
  for (int q = 0; q < kWgCols; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
  const bool do_bias = cg == 0 && (!C.swap || rt == 0);
  int b = (int)((w0 + kk) / V), n = (int)((w0 + kk) - (int64_t)b * V);
  const float* sx = saved + (size_t)layer * terms;
  for (int64_t t = w0; t < w1; t += 4 * kWgUnroll) {
    float ra[kWgUnroll], cb[kWgUnroll][kWgCols];
#pragma unroll
    for (int u = 0; u < kWgUnroll; ++u) {
      const bool ok = t + 4 * u + kk < w1;
      const int bb = ok ? b : 0, nn = ok ? n : 0;
      const float* sb = store + ((size_t)ll * A.B + bb) * PL * V * 4;
      const Site<DIM> s = site_of<DIM>(lat, nn);
      const int par = parity_of<DIM>(s);
      float v;
      if (row_x)
        v = par == fpar ? sx[(size_t)bb * V + nn] : 0.f;
      else
        v = sb[roff + 4 * nn];
      ra[u] = ok && rok ? v : 0.f;
#pragma unroll
      for (int q = 0; q < kWgCols; ++q) {
        const int mm = nbr_site<DIM>(lat, s, ent[q]);
        if (col_x)
          v = ((par ^ (ent[q] >> 12)) & 1) == fpar ? sx[(size_t)bb * V + mm] : 0.f;
        else
          v = sb[coff[q] + 4 * mm];
        cb[u][q] = ok && cok[q] ? v : 0.f;
      }
      n += 4;
      while (n >= V) n -= V, ++b;
    }
#pragma unroll
    for (int u = 0; u < kWgUnroll; ++u) {
      if (do_bias) bias += (double)(C.swap ? cb[u][0] : ra[u]);
      const double da = (double)opnd<BF16>(ra[u]);
#pragma unroll
      for (int q = 0; q < kWgCols; ++q)
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(da, (double)opnd<BF16>(cb[u][q]), acc[q], 0, 0, 0);
    }
  }
  double* out = partial + ((size_t)blockIdx.y * A.layers + ll) * d.P_layer;
#pragma unroll
  for (int q = 0; q < kWgCols; ++q) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) red[w][lane][k] = acc[q][k];
    __syncthreads();
    // thread (lane, w) sums register w of the four waves in order: row 4 w + lane / 16
    const double v = ((red[0][lane][w] + red[1][lane][w]) + red[2][lane][w]) + red[3][lane][w];
    const int rr = rt * 16 + 4 * w + kk;
    if (rr < C.rows && cok[q]) {
      const int f = (cg * kWgCols + q) * 16 + m, tap = f / C.cc, ch = f - tap * C.cc;
      const int co = C.swap ? ch : rr, ci = C.swap ? rr : ch;
      out[d.offW[i] + (co * d.cin[i] + ci) * d.T + tap] = v;
    }
  }
  if (do_bias) {
    redb[w][lane] = bias;
    __syncthreads();
    // rows: channel rt * 16 + m of the row operand; displaced g: the channels of tap 0
    const int ch = C.swap ? cch[0] : row;
    const bool ok = C.swap ? m < C.cc : rok;
    if (w == 0 && kk == 0 && ok) {
      double s = 0.0;
      for (int ww = 0; ww < 4; ++ww)
        for (int k = 0; k < 4; ++k) s += redb[ww][k * 16 + m];
      out[d.offb[i] + ch] = s;
    }
  }
}

// g_params of the group's layers: the chunks' partials summed in order, or, of SLICES waves
// each a share of the chunks in order, then the shares (batch-norm gammas and betas, written
// elsewhere, are left alone).  256 chunks of a few parameters: 10 us by one thread, 5 so.
constexpr int kRedChunks = 64;
template <int SLICES>
__global__ void __launch_bounds__(SLICES > 1 ? 64 * SLICES : 256) kg_reduce(NetDev d, int n, int chunks,
                                                                            const double* __restrict__ partial,
                                                                            float* __restrict__ out) {
  __shared__ double sh[SLICES][64];
  const int col = threadIdx.x & 63, sl = SLICES > 1 ? threadIdx.x >> 6 : 0;
  const int p = SLICES > 1 ? blockIdx.x * 64 + col : blockIdx.x * blockDim.x + threadIdx.x;
  const int c0 = chunks * sl / SLICES, c1 = chunks * (sl + 1) / SLICES;
  double acc = 0.0;
  if (p < n) {
#pragma unroll 8
    for (int c = c0; c < c1; ++c) acc += partial[(size_t)c * n + p];
  }
  if constexpr (SLICES > 1) {
    sh[sl][col] = acc;
    __syncthreads();
    if (sl > 0) return;
#pragma unroll
    for (int k = 1; k < SLICES; ++k) acc += sh[k][col];
  }
  if (p >= n) return;
  if (d.bn) {
    const int r = p % d.P_layer;
    for (int i = 0; i + 1 < d.n_conv; ++i)
      if (r >= d.offg[i] && r < d.offg[i] + 2 * d.cout[i]) return;
  }
  out[p] = (float)acc;
}

// g_z = g_x - g_logq z (d log r / dz = -z); g_logq per sample if g_logq_vec is given.
__global__ void __launch_bounds__(256) kg_gz(int64_t n, const float* __restrict__ gx, const float* __restrict__ z,
                                             float g_logq, const double* __restrict__ g_logq_vec, int64_t V,
                                             float* __restrict__ gz) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gl = g_logq_vec ? (float)g_logq_vec[i / V] : g_logq;
  gz[i] = gx[i] - gl * z[i];
}

// ---- host ------------------------------------------------------------------------

inline unsigned blocks(int64_t n, int per = 256) { return (unsigned)((n + per - 1) / per); }

// Workgroups of the weight-gradient launch: enough chunks of the (sample, site) terms to
// give every CU about four workgroups, each chunk at least 256 terms.
struct WgPlan {
  WgArgs a;
  size_t partial_bytes;
};
WgPlan wgrad_plan(const NetDev& d, int B, int layers, int planes) {
  WgPlan p{};
  WgArgs& a = p.a;
  const int n = d.n_conv;
  int job = 0;
  for (int i = 0; i < n; ++i) {
    WgConv& c = a.c[i];
    const int ci = d.cin[i], co = d.cout[i];
    const int direct = cdiv(co, 16) * cdiv(cdiv(d.T * ci, 16), kWgCols);
    const int swapped = cdiv(ci, 16) * cdiv(cdiv(d.T * co, 16), kWgCols);
    c.swap = co <= 16 && swapped < direct;  // (co: the bias sums sit in one column tile)
    c.rows = c.swap ? ci : co;
    c.cc = c.swap ? co : ci;
    c.ncols = d.T * c.cc;
    c.rt = cdiv(c.rows, 16);
    c.groups = cdiv(cdiv(c.ncols, 16), kWgCols);
    c.gplane = i + 1 < n ? d.hplanes + d.hplane[i] : 2 * d.hplanes;
    c.uplane = i > 0 ? d.hplane[i - 1] : 0;
    c.gseq = d.mode == kSeq && i + 1 < n;
    c.useq = d.mode == kSeq && i > 0;
    c.job0 = job;
    job += c.rt * c.groups;
  }
  a.jobs = job;
  a.layers = layers;
  a.planes = planes;
  a.B = B;
  const int64_t terms = (int64_t)B * d.lat.V;
  int64_t want = std::max<int64_t>(1, 1024 / ((int64_t)job * layers));
  want = std::min<int64_t>(want, std::max<int64_t>(1, terms / 256));
  a.per = ((terms + want - 1) / want + 15) / 16 * 16;
  a.chunks = (int)((terms + a.per - 1) / a.per);
  p.partial_bytes = sizeof(double) * (size_t)a.chunks * layers * d.P_layer;
  return p;
}

// f(std::true_type) or f(std::false_type), and of two conditions.
template <class F>
int32_t with_lf(bool lf, F&& f) {
  return lf ? f(std::true_type{}) : f(std::false_type{});
}
template <class F>
int32_t with_lf(bool lf, bool few, F&& f) {
  return with_lf(lf, [&](auto l) { return with_lf(few, [&](auto w) { return f(l, w); }); });
}

template <int MODE>
void prep(const NetDev& d, const float* params, int layers, int f0, int count, u32x4* frags, hipStream_t st) {
  hipLaunchKernelGGL((kg_prep<MODE>), dim3(blocks((int64_t)layers * count * 64)), dim3(256), 0, st, d, params, layers,
                     f0, count, frags);
}

#define LFS_TRY(x)                            \
  do {                                        \
    const int32_t s_ = (x);                   \
    if (s_ != LFS_OK) return s_;              \
  } while (0)

// Layers whose activations and gradients are kept at once for the weight gradients: as
// many as fit 320 MB; compared at one shape only.  (50 samples of 12^3, 12 layers in one weight-gradient launch or in two
// of 192 MB each, which the last-level cache holds: 591 us or 626.)
int layer_group(const NetDev& d, int B, int planes) {
  const size_t per = (size_t)B * planes * d.lat.V * 16;
  return (int)std::max<size_t>(1, std::min<size_t>(d.N, ((size_t)320 << 20) / per));
}
// The kernels read and write the workspace 16 bytes at a time; a caller's may start
// anywhere, so its first bytes up to the next 16-byte boundary are left unused.
constexpr size_t kWsAlign = 16;
char* aligned_ws(char* ws, size_t* bytes) {
  const size_t skip = (kWsAlign - (uintptr_t)ws % kWsAlign) % kWsAlign;
  *bytes = *bytes > skip ? *bytes - skip : 0;
  return ws + skip;
}

}  // namespace
}  // namespace lfs
