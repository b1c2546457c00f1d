// Convolutions of any s/t network on any lattice as implicit GEMMs on the
// matrix cores (sizes at run time): descriptors, weight fragments, operand
// gathers and the accumulation chains shared by the general kernels.
//
// Activations are FP32 "quad planes": four channels of site n lie at plane q, floats
// 4n .. 4n + 3 (channels past the width are stored as zeros), so sixteen lanes reading
// one quad of sixteen sites touch consecutive bytes.
//
// Order of a forward convolution's sum.  v_mfma_f32_16x16x4_f32 adds its four products
// to the accumulator one after the other, each by a fused multiply-add (k = 0 first), so
// the order of a sum is what the fragments make it:
//   Seq   (FP32, the default network) bias, then taps, channels fastest, one at a time
//   Tree  (FP32, any other) eight sums over the (tap, channel) pairs q = 0, 1, .. with
//         q mod 8 = 0 .. 7, added as ((0+4) + (2+6)) + ((1+5) + (3+7)), then the bias
//   Bf16  v_mfma_f32_16x16x32_bf16 on operands rounded as they are gathered
// The first two are the orders that direct convolutions (one thread, or eight lanes, per
// output) have, so the fields, and with them the signs the backward's LeakyReLU sees, are
// those of such kernels bit for bit.  Data gradients have no order to keep: FP32 takes four
// sums, one per MFMA of a block.
//
// A K block is what a lane group's operand loads bring: 16 k in Seq and in the transposed
// convolutions, 32 in Tree and Bf16.  Seq needs channels j, 4 + j, 8 + j, .. of one tap in
// lane group j, so with it planes hold channels in that order (chan_of).
#pragma once

#include "fused_common.hpp"
#include "lfs_internal.hpp"

namespace lfs {
namespace net {

using fused::bf16x8;
using fused::f32x4;
using fused::pack_bf16;
using fused::u32x2;
using fused::u32x4;
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kMaxConv = LFS_MAX_HIDDEN + 1;

inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// x / d for 0 <= x < 2^32 / d by one high multiplication: with m = ceil(2^32 / d)
// the error x (m d - 2^32) / (2^32 d) stays below 1 / d (x < 2^19, d < 2^13 here).
struct Magic {
  uint32_t m;
  int d;
};
inline Magic magic(int d) { return Magic{(uint32_t)((0x100000000ull + (uint64_t)d - 1) / (uint64_t)d), d}; }
__device__ __forceinline__ int fdiv(int x, const Magic& g) {
  return g.d == 1 ? x : (int)__umulhi((uint32_t)x, g.m);
}

struct Lat {
  int L, V;
  Magic dL, dLL, dH, dV;  // L, L * L, L / 2, V (lattices that live in LDS)
};

enum Mode { kSeq, kTree, kBf16 };

// Channel held by element e of plane pl of an activation of `width` channels, and back.
__host__ __device__ inline int chan_of(bool seq, int width, int pl, int e) {
  if (!seq) return 4 * pl + e;
  return width == 8 ? 4 * (e & 1) + 2 * pl + (e >> 1) : 16 * (pl >> 2) + 4 * e + (pl & 3);
}
__host__ __device__ inline void place_of(bool seq, int width, int c, int& pl, int& e) {
  if (!seq) {
    pl = c >> 2;
    e = c & 3;
  } else if (width == 8) {
    pl = (c & 3) >> 1;
    e = 2 * (c & 1) + (c >> 2);
  } else {
    pl = 4 * (c >> 4) + (c & 3);
    e = (c >> 2) & 3;
  }
}

// One convolution in one direction.  Forward: rows are output channels and K runs
// over the input channels; transposed: rows are input channels, K over output ones.
struct ConvDir {
  int rows, nct;   // rows and 16-row tiles
  Magic dnct;
  int ck, nq;      // channels of K and quads per tap
  Magic dnq, dck;
  int nb, fpb;     // K blocks, fragments (1 KB) per block
  int off;         // first fragment of the layer's fragments; per row tile nb fpb + 1 of
                   // them, the first holding the bias (zeros when transposed)
  __host__ __device__ int per_ct() const { return nb * fpb + 1; }
};

struct NetDev {
  int dim, N, n_conv, K, T, parity0, final_tanh, mode;
  Magic dK;
  int wide;  // K / 2 >= L: tap offsets need reducing modulo L
  Lat lat;
  int cin[kMaxConv], cout[kMaxConv];
  int offW[kMaxConv], offb[kMaxConv];
  int P_layer;
  ConvDir f[kMaxConv], t[kMaxConv];
  int frags_fwd, frags_all;  // fragments per layer: forward only, both directions
  int hplane[kMaxConv];      // first plane of hidden activation i (hidden planes in order)
  int hplanes;               // planes of all hidden activations
  int bn;                    // batch norm: gamma (beta at + cout) of hidden convolution i at offg[i]
  int offg[LFS_MAX_HIDDEN];
};

inline NetDev make_net(const FlowGeom& g) {
  NetDev d{};
  d.dim = g.dim;
  d.N = g.N;
  d.n_conv = g.n_conv;
  d.K = g.K;
  d.T = g.T;
  d.dK = magic(g.K);
  d.wide = g.K / 2 >= g.L;
  d.parity0 = g.parity0;
  d.final_tanh = g.final_tanh;
  d.mode = g.bf16() ? kBf16 : g.net_default ? kSeq : kTree;
  d.lat = Lat{g.L, g.V, magic(g.L), magic(g.L * g.L), magic(g.L / 2), magic(g.V)};
  d.P_layer = (int)g.P_layer;
  d.bn = g.bn;
  int off = 0;
  for (int dir = 0; dir < 2; ++dir) {
    for (int i = 0; i < g.n_conv; ++i) {
      ConvDir& c = dir ? d.t[i] : d.f[i];
      c.rows = dir ? g.cin[i] : g.cout[i];
      c.nct = cdiv(c.rows, 16);
      c.dnct = magic(c.nct);
      c.ck = dir ? g.cout[i] : g.cin[i];
      c.dck = magic(c.ck);
      const bool first = dir == 0 && i == 0;
      c.nq = first ? 1 : cdiv(c.ck, 4);
      c.dnq = magic(c.nq);
      c.fpb = dir == 0 && d.mode == kTree ? 2 : 1;
      // Tree runs over the (tap, channel) pairs themselves, the others over quads
      const int quads = first ? cdiv(g.T, 4) : g.T * c.nq;
      c.nb = dir == 0 && d.mode == kTree ? cdiv(g.T * c.ck, 32) : cdiv(quads, d.mode == kBf16 ? 8 : 4);
      c.off = off;
      off += c.nct * c.per_ct();
    }
    if (dir == 0) d.frags_fwd = off;
  }
  d.frags_all = off;
  for (int i = 0; i < g.n_conv; ++i) {
    d.cin[i] = g.cin[i];
    d.cout[i] = g.cout[i];
    d.offW[i] = (int)g.offW[i];
    d.offb[i] = (int)g.offb[i];
    d.hplane[i] = d.hplanes;
    if (i + 1 < g.n_conv) d.hplanes += cdiv(g.cout[i], 4);
    if (g.bn && i + 1 < g.n_conv) d.offg[i] = (int)g.offg[i];
  }
  return d;
}

// Channel of fragment row `row` of convolution i (rows follow the output planes).
__device__ __forceinline__ int row_chan(const NetDev& d, int i, bool tr, int row) {
  const bool hidden = tr ? i > 0 : i + 1 < d.n_conv;
  return chan_of(d.mode == kSeq && hidden, tr ? d.cin[i] : d.cout[i], row >> 2, row & 3);
}

// Weight W[co][ci][tap] at fragment row `row` and element r of lane group j in fragment f
// (block f / fpb) of a row tile; 0 past the ends.
template <int MODE>
__device__ __forceinline__ float w_at(const NetDev& d, const float* pl, int i, bool tr, int row, int f, int j, int r) {
  const ConvDir& c = tr ? d.t[i] : d.f[i];
  if (row >= c.rows) return 0.f;
  int tap, ch;
  if (!tr && MODE == kTree) {
    const int q = 8 * (4 * (f >> 1) + j) + 4 * (f & 1) + r;
    tap = q / c.ck;
    ch = q - tap * c.ck;
  } else if (!tr && i == 0) {
    tap = MODE == kSeq ? 16 * f + 4 * r + j : 4 * (4 * f + j) + r;  // (Bf16: f counts quads of four groups)
    ch = 0;
  } else if (!tr && MODE == kSeq && c.ck == 8) {
    tap = 2 * f + (r >> 1);
    ch = 4 * (r & 1) + j;
  } else {
    const int q = 4 * f + j;
    tap = q / c.nq;
    ch = chan_of(MODE == kSeq && (tr ? i + 1 < d.n_conv : true), c.ck, q - tap * c.nq, r);
  }
  if (tap >= d.T || ch >= c.ck) return 0.f;
  const int rc = row_chan(d, i, tr, row);
  const int co = tr ? ch : rc, ci = tr ? rc : ch;
  return pl[d.offW[i] + (co * d.cin[i] + ci) * d.T + tap];
}

// Lane l's 16 bytes of fragment (ct, f) of convolution i: f = -1 the bias of rows
// 4j .. 4j + 3 (forward), else weights.
template <int MODE>
__device__ __forceinline__ u32x4 frag_entry(const NetDev& d, const float* pl, int i, bool tr, int ct, int f, int l) {
  const int j = l >> 4, m = l & 15;
  u32x4 o{0u, 0u, 0u, 0u};
  if (f < 0) {
    if (!tr)
      for (int r = 0; r < 4; ++r) {
        const int row = ct * 16 + 4 * j + r;
        if (row < d.cout[i]) o[r] = __float_as_uint(pl[d.offb[i] + row_chan(d, i, false, row)]);
      }
    return o;
  }
  const int row = ct * 16 + m;
  if constexpr (MODE == kBf16) {
    // lane group j of block f holds quads 8 f + 2 j and 8 f + 2 j + 1: as quads of four
    // lane groups, (2 f + (j >> 1), 2 (j & 1) + h)
    for (int h = 0; h < 2; ++h) {
      const int f4 = 2 * f + (j >> 1), j4 = 2 * (j & 1) + h;
      o[2 * h] = pack_bf16(w_at<MODE>(d, pl, i, tr, row, f4, j4, 0), w_at<MODE>(d, pl, i, tr, row, f4, j4, 1));
      o[2 * h + 1] = pack_bf16(w_at<MODE>(d, pl, i, tr, row, f4, j4, 2), w_at<MODE>(d, pl, i, tr, row, f4, j4, 3));
    }
  } else {
    for (int r = 0; r < 4; ++r) o[r] = __float_as_uint(w_at<MODE>(d, pl, i, tr, row, f, j, r));
  }
  return o;
}

// A operands of one convolution: its fragments, row tile by row tile.
struct Weights {
  const u32x4* frags;
  int per_ct, lane;
  __device__ __forceinline__ u32x4 at(int ct, int f) const {  // f = -1: bias
    return frags[(ct * per_ct + f + 1) * 64 + lane];
  }
  // element e of the lane's 16 bytes
  __device__ __forceinline__ float elem(int ct, int f, int e) const {
    return reinterpret_cast<const float*>(frags + (ct * per_ct + f + 1) * 64 + lane)[e];
  }
};

// ---- lattice coordinates and gathers -------------------------------------------

template <int DIM>
struct Site {
  int c[DIM];
};

template <int DIM>
__device__ __forceinline__ Site<DIM> site_of(const Lat& a, int n) {
  Site<DIM> s;
  if constexpr (DIM == 2) {
    s.c[0] = fdiv(n, a.dL);
    s.c[1] = n - s.c[0] * a.L;
  } else {
    s.c[0] = fdiv(n, a.dLL);
    const int r = n - s.c[0] * a.L * a.L;
    s.c[1] = fdiv(r, a.dL);
    s.c[2] = r - s.c[1] * a.L;
  }
  return s;
}

template <int DIM>
__device__ __forceinline__ int parity_of(const Site<DIM>& s) {
  int p = s.c[0] + s.c[1];
  if constexpr (DIM == 3) p += s.c[2];
  return p & 1;
}

// The a-th site (row-major) among the V / 2 sites of parity par.
template <int DIM>
__device__ __forceinline__ int half_site(const Lat& g, int a, int par) {
  const int row = fdiv(a, g.dH), i = a - row * (g.L >> 1);
  int lead = row;
  if constexpr (DIM == 3) {
    const int z = fdiv(row, g.dL);
    lead = z + row - z * g.L;
  }
  return row * g.L + 2 * i + ((par + lead) & 1);
}

// (c mod L) for -L < c < 2 L: a value out of range is huge, or larger than its corrected
// form, as an unsigned number.
__device__ __forceinline__ int wrap_c(int c, int L) {
  uint32_t v = (uint32_t)c;
  v = min(v, v + (uint32_t)L);
  return (int)min(v, v - (uint32_t)L);
}

// Tap table entry: offsets + 8 in 4-bit fields (axis 0 lowest; reduced modulo L, so that
// one wrap each way is enough for kernels wider than the lattice), the parity of |delta|_1
// in bit 12, bit 31 set past the last tap (whose operand is the site's own value, replaced
// by zero).
constexpr int kTabPad = (int)0x80000000;

template <int DIM>
__device__ __forceinline__ int tap_entry(const NetDev& d, int tap, int sign) {
  int e = 0, p = 0, t = tap;
#pragma unroll
  for (int mu = DIM - 1; mu >= 0; --mu) {
    const int q = fdiv(t, d.dK);
    int o = t - q * d.K - (d.K >> 1);
    if (d.wide) o %= d.lat.L;
    e |= (sign * o + 8) << (4 * mu);
    p += o;
    t = q;
  }
  return e | ((p & 1) << 12);
}

template <int DIM>
__device__ __forceinline__ int site_entry() {
  return DIM == 2 ? 0x88 : 0x888;  // no offset
}

template <int DIM>
__device__ __forceinline__ int nbr_site(const Lat& a, const Site<DIM>& s, int e) {
  int r = wrap_c(s.c[0] + (e & 15) - 8, a.L);
  r = r * a.L + wrap_c(s.c[1] + ((e >> 4) & 15) - 8, a.L);
  if constexpr (DIM == 3) r = r * a.L + wrap_c(s.c[2] + ((e >> 8) & 15) - 8, a.L);
  return r;
}

// Tap table of the lattice into LDS: entry t for the site n + sign delta_t, then padding.
template <int DIM>
__device__ __forceinline__ void build_tab(const NetDev& d, int sign, int* tab) {
  for (int t = threadIdx.x; t <= d.T; t += blockDim.x)
    tab[t] = t < d.T ? tap_entry<DIM>(d, t, sign) : site_entry<DIM>() | kTabPad;
}

// Neighbour table in LDS, for samples that live there: site n + delta_t at [t][n], and a
// row T of entries V, the zero site that follows every plane and the field.  The
// transposed convolution's neighbour n - delta_t is row T - 1 - t.
template <int DIM>
__device__ __forceinline__ void build_nbr(const NetDev& d, uint16_t* nb) {
  const Lat& lat = d.lat;
  for (int k = threadIdx.x; k < (d.T + 1) * lat.V; k += blockDim.x) {
    const int t = fdiv(k, lat.dV), n = k - t * lat.V;
    nb[k] = (uint16_t)(t < d.T ? nbr_site<DIM>(lat, site_of<DIM>(lat, n), tap_entry<DIM>(d, t, 1)) : lat.V);
  }
}

// Keeps a float where the mask is all ones, zero where it is 0 (no branch, whatever the
// value).
__device__ __forceinline__ float masked(float v, int mask) { return __uint_as_float(__float_as_uint(v) & (uint32_t)mask); }

// ---- operand readers ---------------------------------------------------------------
// A reader gives the operands of the lane's site: val(t, pl, e) element e of plane pl at tap
// t (the field: pl = e = 0), quad(t, pl) and pair(t, pl, h) whole and half planes.  Taps at
// or past T read zeros.

// Beyond the LDS: neighbours by arithmetic (tab: build_tab), planes ps floats apart.
template <int DIM>
struct FarPlanes {
  const Lat* lat;
  const int* tab;
  const float* base;
  int ps, T;
  Site<DIM> s;
  __device__ __forceinline__ float val(int t, int pl, int e) const {
    const int x = tab[min(t, T)];
    return masked(base[pl * ps + 4 * nbr_site<DIM>(*lat, s, x) + e], ~(x >> 31));
  }
  __device__ __forceinline__ f32x4 quad(int t, int pl) const {
    const int x = tab[min(t, T)];
    f32x4 v = *reinterpret_cast<const f32x4*>(base + pl * ps + 4 * nbr_site<DIM>(*lat, s, x));
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = masked(v[r], ~(x >> 31));
    return v;
  }
  __device__ __forceinline__ f32x2 pair(int t, int pl, int h) const {
    const int x = tab[min(t, T)];
    f32x2 v = *reinterpret_cast<const f32x2*>(base + pl * ps + 4 * nbr_site<DIM>(*lat, s, x) + 2 * h);
#pragma unroll
    for (int r = 0; r < 2; ++r) v[r] = masked(v[r], ~(x >> 31));
    return v;
  }
};

template <int DIM>
struct FarField {
  const Lat* lat;
  const int* tab;
  const float* x;
  int T, flip;  // flip: the site's parity ^ the frozen parity
  Site<DIM> s;
  __device__ __forceinline__ float val(int t, int, int) const {
    const int e = tab[min(t, T)];
    return masked(x[nbr_site<DIM>(*lat, s, e)], ~(e >> 31) & (((flip ^ (e >> 12)) & 1) - 1));
  }
};

// In LDS: neighbours from the table (nb: the site's column; row T: the zero site that
// follows every plane and the field).  REV: n - delta_t.
template <bool REV>
struct LdsPlanes {
  const uint16_t* nb;
  const float* base;
  int V, ps, T;
  __device__ __forceinline__ const float* at(int t, int pl) const {
    const int row = REV ? (t < T ? T - 1 - t : T) : min(t, T);
    return base + pl * ps + 4 * nb[row * V];
  }
  __device__ __forceinline__ float val(int t, int pl, int e) const { return at(t, pl)[e]; }
  __device__ __forceinline__ f32x4 quad(int t, int pl) const { return *reinterpret_cast<const f32x4*>(at(t, pl)); }
  __device__ __forceinline__ f32x2 pair(int t, int pl, int h) const {
    return *reinterpret_cast<const f32x2*>(at(t, pl) + 2 * h);
  }
};

struct LdsField {
  const uint16_t* nb;
  const float* x;
  int V, T, flip;
  const int* odd;  // per tap, the parity of |delta|_1 (0 past the last)
  __device__ __forceinline__ float val(int t, int, int) const {
    const int r = min(t, T), m = nb[r * V];
    return x[(odd[r] ^ flip) ? V : m];  // an active site reads the zero that follows the field
  }
};

// The four channels (FIRST: taps) of quad q of a convolution's K.
template <bool FIRST, class R>
__device__ __forceinline__ f32x4 quad_of(const R& rd, const ConvDir& c, int q) {
  if constexpr (FIRST) {
    return f32x4{rd.val(4 * q, 0, 0), rd.val(4 * q + 1, 0, 0), rd.val(4 * q + 2, 0, 0), rd.val(4 * q + 3, 0, 0)};
  } else {
    const int t = fdiv(q, c.dnq);
    return rd.quad(t, q - t * c.nq);
  }
}

// The lane's operand of block b: lane group j of a transposed convolution (FP32) or of a
// Seq one.
template <int MODE, bool TR, bool FIRST, class R>
__device__ __forceinline__ u32x4 operand(const R& rd, const ConvDir& c, int j, int b) {
  if constexpr (MODE == kBf16) {
    const f32x4 u = quad_of<FIRST>(rd, c, 8 * b + 2 * j), v = quad_of<FIRST>(rd, c, 8 * b + 2 * j + 1);
    return u32x4{pack_bf16(u[0], u[1]), pack_bf16(u[2], u[3]), pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
  } else if constexpr (!TR && FIRST) {  // Seq: taps 16 b + 4 r + j
    return __builtin_bit_cast(u32x4, f32x4{rd.val(16 * b + j, 0, 0), rd.val(16 * b + 4 + j, 0, 0),
                                           rd.val(16 * b + 8 + j, 0, 0), rd.val(16 * b + 12 + j, 0, 0)});
  } else {
    if constexpr (!TR)
      if (c.ck == 8) {  // Seq: channels j and 4 + j of taps 2 b and 2 b + 1
        const f32x2 u = rd.pair(2 * b, j >> 1, j & 1), v = rd.pair(2 * b + 1, j >> 1, j & 1);
        return __builtin_bit_cast(u32x4, f32x4{u[0], u[1], v[0], v[1]});
      }
    return __builtin_bit_cast(u32x4, quad_of<false>(rd, c, 4 * b + j));
  }
}

// ---- accumulation chains -----------------------------------------------------------

// Sum over K blocks [b0, b1) on top of init: transposed, Seq and Bf16 convolutions.  U
// blocks' operands are in flight; PIPE: the next U are fetched while the current ones are
// multiplied (operands from beyond the LDS).  kmax: channels of a one-quad convolution
// (MFMA r of a block takes channel r of every lane group's quad; past them all is zero).
template <int MODE, bool TR, bool FIRST, int U, bool PIPE, class R>
__device__ __forceinline__ f32x4 chain(const R& rd, const ConvDir& c, const Weights& W, int ct, int j, int b0, int b1,
                                       const f32x4& init) {
  constexpr bool FOUR = MODE != kBf16 && TR;  // four sums
  f32x4 s[FOUR ? 4 : 1];
  s[0] = init;
  if constexpr (FOUR) s[1] = s[2] = s[3] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int kmax = TR && c.nq == 1 ? c.ck : 4, last = b1 - 1;
  auto mul = [&](const u32x4& a, const u32x4& b) {
    if constexpr (MODE == kBf16) {
      s[0] = fused::mfma(fused::as_bf16x8(a), fused::as_bf16x8(b), s[0]);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r < 2 || r < kmax)
          s[FOUR ? r : 0] = fused::mfma(__uint_as_float(a[r]), __uint_as_float(b[r]), s[FOUR ? r : 0]);
    }
  };
  u32x4 a[U], b[U];
  if constexpr (!PIPE) {
    for (int k = b0; k < b1; k += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = min(k + u, last);
        a[u] = W.at(ct, q);
        b[u] = operand<MODE, TR, FIRST>(rd, c, j, q);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u < b1) mul(a[u], b[u]);
    }
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = min(b0 + u, last);
      a[u] = W.at(ct, q);
      b[u] = operand<MODE, TR, FIRST>(rd, c, j, q);
    }
    for (int k = b0; k < b1; k += U) {
      u32x4 an[U], bn[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = min(k + U + u, last);
        an[u] = W.at(ct, q);
        bn[u] = operand<MODE, TR, FIRST>(rd, c, j, q);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u < b1) mul(a[u], b[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = an[u], b[u] = bn[u];
    }
  }
  if constexpr (FOUR) return (s[0] + s[1]) + (s[2] + s[3]);
  return s[0];
}

// The eight elements of lane group j of Tree block b: (tap, channel) pairs 8 (4 b + j) ..
// + 7, as two quads (h = 0, 1), or element e of quad h.
template <bool FIRST, class R>
__device__ __forceinline__ f32x4 tree_quad(const R& rd, const ConvDir& c, int j, int b, int h) {
  const int Q = 2 * (4 * b + j) + h;
  if constexpr (FIRST) {
    return quad_of<true>(rd, c, Q);
  } else if ((c.ck & 3) == 0) {
    return quad_of<false>(rd, c, Q);
  } else {  // quads that straddle taps
    f32x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = fdiv(4 * Q + r, c.dck), ch = 4 * Q + r - t * c.ck;
      v[r] = rd.val(t, ch >> 2, ch & 3);
    }
    return v;
  }
}
template <bool FIRST, class R>
__device__ __forceinline__ float tree_elem(const R& rd, const ConvDir& c, int j, int b, int h, int e) {
  const int q = 8 * (4 * b + j) + 4 * h + e;
  if constexpr (FIRST) {
    return rd.val(q, 0, 0);
  } else {
    const int t = fdiv(q, c.dck), ch = q - t * c.ck;
    return rd.val(t, ch >> 2, ch & 3);
  }
}

// Tree convolution without its bias; SPLIT: only the sums part and part + 4 (the other
// parts are other waves', see tree_join).
template <bool FIRST, bool SPLIT, class R>
__device__ __forceinline__ f32x4 tree(const R& rd, const ConvDir& c, const Weights& W, int ct, int j, int part) {
  const f32x4 zero{0.f, 0.f, 0.f, 0.f};
  if constexpr (SPLIT) {
    f32x4 s0 = zero, s1 = zero;
    for (int b0 = 0; b0 < c.nb; b0 += 2) {
      float a[2][2], v[2][2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int b = min(b0 + u, c.nb - 1);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          a[u][h] = W.elem(ct, 2 * b + h, part);
          v[u][h] = tree_elem<FIRST>(rd, c, j, b, h, part);
        }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (b0 + u < c.nb) {
          s0 = fused::mfma(a[u][0], v[u][0], s0);
          s1 = fused::mfma(a[u][1], v[u][1], s1);
        }
    }
    return s0 + s1;
  } else {
    f32x4 s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e] = zero;
    for (int b = 0; b < c.nb; ++b) {
      u32x4 a[2];
      f32x4 v[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        a[h] = W.at(ct, 2 * b + h);
        v[h] = tree_quad<FIRST>(rd, c, j, b, h);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] = fused::mfma(__uint_as_float(a[e >> 2][e & 3]), v[e >> 2][e & 3], s[e]);
    }
    return ((s[0] + s[4]) + (s[2] + s[6])) + ((s[1] + s[5]) + (s[3] + s[7]));
  }
}

}  // namespace net
}  // namespace lfs
