// Convolutions of any s/t network on any lattice as implicit GEMMs on the
// matrix cores (sizes at run time): descriptors, weight fragments, operand
// gathers and the accumulation chains shared by the general kernels.
//
// Activations are FP32 "quad planes": four channels of site n lie at plane q, floats
// 4n .. 4n + 3 (channels past the width are stored as zeros), so sixteen lanes reading
// one quad of sixteen sites touch consecutive bytes.
//
// Order of a convolution's sum, in both directions.  v_mfma_f32_16x16x4_f32 adds its four
// products to the accumulator one after the other, each by a fused multiply-add (k = 0
// first), so the order of a sum is what the fragments make it:
//   Seq   (FP32, the default network) bias, then taps, channels fastest, one at a time (the
//         last one's transpose: tap by tap, its two products added to each other first)
//   Tree  (FP32, any other) eight sums over the (tap, channel) pairs q = 0, 1, .. with
//         q mod 8 = 0 .. 7, added as ((0+4) + (2+6)) + ((1+5) + (3+7)), then the bias
//   Bf16  v_mfma_f32_16x16x32_bf16 on operands rounded as they are gathered
// The first two are the orders that direct convolutions (one thread, or eight lanes, per
// output) have, so the fields, and with them the signs the backward's LeakyReLU sees, are
// those of such kernels bit for bit, and the data gradients too: an optimizer step that
// follows gradients a bit away moves the parameters, and in the next step an activation next
// to zero may change its sign.
//
// A K block is what a lane group's operand loads bring: 16 k in Seq, 32 in Tree and Bf16.
// Seq needs channels j, 4 + j, 8 + j, .. of one tap in lane group j, so with it planes hold
// channels in that order (chan_of).
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
  int dq, rq;      // quads a lane advances per block (8, or 4), as taps and planes
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
      c.fpb = d.mode == kTree ? 2 : 1;
      // Tree runs over the (tap, channel) pairs themselves, the others over quads
      const int quads = first ? cdiv(g.T, 4) : g.T * c.nq;
      c.nb = d.mode == kTree ? cdiv(g.T * c.ck, 32) : cdiv(quads, d.mode == kBf16 ? 8 : 4);
      const int inc = d.mode == kSeq ? 4 : 8;
      c.dq = inc / c.nq;
      c.rq = inc % c.nq;
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
  if (MODE == kTree) {
    const int q = 8 * (4 * (f >> 1) + j) + 4 * (f & 1) + r;
    tap = q / c.ck;
    ch = q - tap * c.ck;
  } else if (!tr && i == 0) {
    tap = MODE == kSeq ? 16 * f + 4 * r + j : 4 * (4 * f + j) + r;  // (Bf16: f counts quads of four groups)
    ch = 0;
  } else if (tr && MODE == kSeq && i + 1 == d.n_conv) {  // Seq: output 1, then output 0 of tap 4 f + r
    if (j > 1) return 0.f;
    tap = 4 * f + r;
    ch = 1 - j;
  } else if (MODE == kSeq && c.ck == 8) {
    tap = 2 * f + (r >> 1);
    ch = 4 * (r & 1) + j;
  } else {
    const int q = 4 * f + j;
    tap = q / c.nq;
    ch = chan_of(MODE == kSeq, c.ck, q - tap * c.nq, r);
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

// A tap's offsets + 8 in 4-bit fields (axis 0 lowest; reduced modulo L, so that one wrap each
// way is enough for kernels wider than the lattice) and the parity of |delta|_1 in bit 12.

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
__device__ __forceinline__ int nbr_site(const Lat& a, const Site<DIM>& s, int e) {
  int r = wrap_c(s.c[0] + (e & 15) - 8, a.L);
  r = r * a.L + wrap_c(s.c[1] + ((e >> 4) & 15) - 8, a.L);
  if constexpr (DIM == 3) r = r * a.L + wrap_c(s.c[2] + ((e >> 8) & 15) - 8, a.L);
  return r;
}

// Neighbour table in LDS, for samples that live there: site n + delta_t in row t, and one
// row of V before and after: V is the zero site that follows the field and every plane,
// which the quads past a convolution's last one read, also in reverse order (the transposed
// convolution's neighbour n - delta_t is in row T - 1 - t).
inline int64_t nbr_bytes(int T, int V) { return 2ll * (T + 2) * V; }
template <int DIM>
__device__ __forceinline__ void build_nbr(const NetDev& d, uint16_t* nb) {
  // a wave per row, a lane per site: the tap is the wave's, a site's coordinates are found once
  // (entry by entry, with four divisions each, a batch-norm step of 144 launches took 940 us
  // instead of 934)
  const Lat& lat = d.lat;
  for (int n = threadIdx.x & 63; n < lat.V; n += 64) {
    const Site<DIM> s = site_of<DIM>(lat, n);
    for (int r = fused::wave_id(); r < d.T + 2; r += blockDim.x >> 6)
      nb[r * lat.V + n] =
          (uint16_t)(r > 0 && r <= d.T ? nbr_site<DIM>(lat, s, tap_entry<DIM>(d, r - 1, 1)) : lat.V);
  }
}

// Keeps a float where the mask is all ones, zero where it is 0 (no branch, whatever the
// value).
__device__ __forceinline__ float masked(float v, int mask) { return __uint_as_float(__float_as_uint(v) & (uint32_t)mask); }

// For samples beyond the LDS, the neighbours n + sign delta_t of kTileSites sites: site k's in
// column k, tap t's in row t, then a row for the quads past the end.  Entries that read zero
// have the top bit set: that row's and, for a field (frozen parity fpar; -1: a plane), the
// active sites'.  site(k) is the k-th site.
constexpr int kTileSites = 64;
constexpr uint32_t kZero = 0x80000000u;
__host__ __device__ inline int tile_table_bytes(int T) { return 4 * (T + 1) * kTileSites; }
template <int DIM, class S>
__device__ __forceinline__ void build_tile(const NetDev& d, int sign, int fpar, uint32_t* nb, S&& site) {
  const int k = threadIdx.x % kTileSites, n = site(k);
  const Site<DIM> s = site_of<DIM>(d.lat, n);
  const int flip = parity_of<DIM>(s) ^ fpar;
  for (int t = fused::wave_id(); t <= d.T; t += blockDim.x / kTileSites) {  // a wave per tap
    uint32_t v = (uint32_t)n | kZero;
    if (t < d.T) {
      const int e = tap_entry<DIM>(d, t, sign);
      v = (uint32_t)nbr_site<DIM>(d.lat, s, e);
      if (fpar >= 0 && ((flip ^ (e >> 12)) & 1)) v |= kZero;
    }
    nb[t * kTileSites + k] = v;
  }
}

// ---- convolutions ------------------------------------------------------------------
// Operands are gathered through a table of neighbours in LDS: of a whole sample that lives
// there (LDS: 16-bit entries, one table for all taps and both directions, zeros kept behind
// the field and the planes), or of a tile of a larger one (32-bit entries, a table per
// launch).  A lane's quads are a fixed number of taps and planes apart from block to block,
// so its place is stepped instead of formed by a division per quad (with a division and 12
// instructions of wrapping per quad, width 16: a hidden convolution of an 8 x 8 sample took
// 6500 clocks against the 1280 of its MFMAs, one of 50 samples of 12^3 41 us; now 3500 and
// 25 us).

// An operand's place: plane (from its element on) and table entry.  What it reads beyond the
// LDS goes through kept() before it is used, and not before: masked where it is loaded, every
// block waited for the loads of the blocks ahead.
template <bool LDS>
struct At {
  const float* plane;
  uint32_t site;
  __device__ __forceinline__ const float* get() const {
    if constexpr (LDS) return plane + 4 * site;
    return plane + 4 * (size_t)(site & ~kZero);
  }
  __device__ __forceinline__ f32x4 quad() const { return *reinterpret_cast<const f32x4*>(get()); }
  __device__ __forceinline__ f32x2 pair() const { return *reinterpret_cast<const f32x2*>(get()); }
};
template <bool LDS>
__device__ __forceinline__ float kept(float v, uint32_t site) {
  return LDS ? v : masked(v, ~((int)site >> 31));
}
template <bool LDS>
__device__ __forceinline__ f32x4 kept(f32x4 v, uint32_t site) {
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = kept<LDS>(v[r], site);
  return v;
}

// The reader of planes `base` (stride ps floats) for the lane's site; nb: the site's column
// of the table at tap 0, rows V entries long.  REV (LDS only): n - delta_t.
template <bool REV, bool LDS>
struct Planes {
  using Entry = std::conditional_t<LDS, uint16_t, uint32_t>;
  using Place = At<LDS>;
  static constexpr bool rev = REV, lds = LDS;
  const Entry* nb;
  const float* base;
  int V, ps, T;
};

template <bool REV, bool LDS>
struct Walk {
  using Entry = typename Planes<REV, LDS>::Entry;
  const Entry* row;
  const Entry* end;  // the row that reads zero
  const float* plane;
  int pl, nq, up, over, rq, ps;  // up: table step of dq taps; over: of one tap
  __device__ __forceinline__ Walk(const Planes<REV, LDS>& r, const ConvDir& c, int q) {
    const int t = fdiv(q, c.dnq);
    pl = q - __mul24(t, c.nq);
    row = r.nb + __mul24(REV ? r.T - 1 - t : t, r.V);
    end = r.nb + (REV ? -1 : r.T) * r.V;
    plane = r.base + pl * r.ps;
    over = REV ? -r.V : r.V;
    up = c.dq * over;
    nq = c.nq;
    rq = c.rq;
    ps = r.ps;
  }
  __device__ __forceinline__ At<LDS> next() {
    const At<LDS> at{plane, *((REV ? row < end : row > end) ? end : row)};
    row += up;
    if (rq != 0) {  // uniform
      pl += rq;
      const bool carry = pl >= nq;
      pl -= carry ? nq : 0;
      plane += (carry ? rq - nq : rq) * ps;
      row += carry ? over : 0;
    }
    return at;
  }
};

// The reader of the masked field (zero at the active sites and past the end).
template <bool LDS>
struct Field {
  static constexpr bool lds = LDS;
  using Entry = typename Planes<false, LDS>::Entry;
  const Entry* nb;
  const float* x;
  int V, T;
  __device__ __forceinline__ uint32_t find(int t) const { return nb[__mul24(min(t, T), V)]; }
  __device__ __forceinline__ float get(uint32_t e) const { return x[LDS ? e : e & ~kZero]; }
};
template <class R>
struct IsField : std::false_type {};
template <bool LDS>
struct IsField<Field<LDS>> : std::true_type {};

// The place of (tap, channel) pair q of planes whose width is no multiple of four.
template <bool REV, bool LDS>
__device__ __forceinline__ At<LDS> pair_at(const Planes<REV, LDS>& r, const ConvDir& c, int q) {
  const int t = fdiv(q, c.dck), ch = q - __mul24(t, c.ck), row = REV ? max(r.T - 1 - t, -1) : min(t, r.T);
  return {r.base + (ch >> 2) * r.ps + (ch & 3), r.nb[row * r.V]};
}

// K blocks [b0, b1): find(b) looks places up, fetch(b, what find gave) reads operands, mul
// multiplies them.  In LDS (AHEAD = 0) the three are one block apart, so neither of the two
// latencies stands between a block's MFMAs and the next one's; beyond it AHEAD blocks are
// found and fetched together, before the AHEAD ones before them are multiplied: a block's
// MFMAs take 128 clocks, its gather from the L2 several times that (width 16, 50 samples of
// 12^3: 31 us with the loads of one block in flight, 25 us with four).  Past the end the last block is found and fetched again (a walk meets the zero
// row) and not multiplied.
template <int AHEAD, class Find, class Fetch, class Mul>
__device__ __forceinline__ void walk_blocks(int b0, int b1, Find&& find, Fetch&& fetch, Mul&& mul) {
  const int last = b1 - 1;
  if constexpr (AHEAD == 0) {
    auto f = find(b0);
    auto v = fetch(b0, f);
    f = find(min(b0 + 1, last));
    for (int b = b0; b < b1; ++b) {
      const auto vn = fetch(min(b + 1, last), f);
      f = find(min(b + 2, last));
      mul(v);
      v = vn;
    }
  } else {
    decltype(find(0)) f[AHEAD];
    decltype(fetch(0, f[0])) v[AHEAD], vn[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) f[u] = find(min(b0 + u, last));
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) v[u] = fetch(min(b0 + u, last), f[u]);
    for (int b = b0; b < b1; b += AHEAD) {
      if (b + AHEAD < b1) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) f[u] = find(min(b + AHEAD + u, last));
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) vn[u] = fetch(min(b + AHEAD + u, last), f[u]);
      }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (u == 0 || b + u < b1) mul(v[u]);
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) v[u] = vn[u];
    }
  }
}

// A lane's index the compiler knows nothing of: what is derived from it in a branch stays
// there, instead of being set up for every branch ahead of the loop over units.
__device__ __forceinline__ int opaque(int j) {
  asm volatile("" : "+v"(j));
  return j;
}

// init + the sum over K blocks [b0, b1): Seq and Bf16 convolutions.
template <int MODE, bool TR, class R>
__device__ __forceinline__ f32x4 chain(const R& rd, const ConvDir& c, const Weights& W, int ct, int j0, int b0, int b1,
                                       const f32x4& init) {
  constexpr bool L = R::lds;
  constexpr int AHEAD = L ? 0 : 4;
  f32x4 s = init;
  auto mul = [&](const u32x4& a, const f32x4& b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) s = fused::mfma(__uint_as_float(a[r]), b[r], s);
  };
  auto mul16 = [&](const u32x4& a, const f32x4& u, const f32x4& v) {
    const u32x4 b{pack_bf16(u[0], u[1]), pack_bf16(u[2], u[3]), pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    s = fused::mfma(fused::as_bf16x8(a), fused::as_bf16x8(b), s);
  };
  const int j = opaque(j0);
  if constexpr (IsField<R>::value) {
    constexpr int NS = MODE == kBf16 ? 8 : 4;
    struct Sites {
      uint32_t n[NS];
    };
    struct Op {
      u32x4 a;
      float v[NS];
      Sites f;
    };
    walk_blocks<AHEAD>(b0, b1, [&](int b) {
      Sites f;
#pragma unroll
      for (int r = 0; r < NS; ++r) f.n[r] = rd.find(MODE == kSeq ? 16 * b + 4 * r + j : 32 * b + 8 * j + r);
      return f;
    }, [&](int b, const Sites& f) {
      Op o{W.at(ct, b), {}, f};
#pragma unroll
      for (int r = 0; r < NS; ++r) o.v[r] = rd.get(f.n[r]);
      return o;
    }, [&](const Op& o) {
      f32x4 v[NS / 4];
#pragma unroll
      for (int r = 0; r < NS; ++r) v[r / 4][r % 4] = kept<L>(o.v[r], o.f.n[r]);
      if constexpr (MODE == kBf16) mul16(o.a, v[0], v[1]);
      else mul(o.a, v[0]);
    });
  } else {
    using P = typename R::Place;
    if constexpr (MODE == kBf16) {
      struct Two {
        P u, v;
      };
      struct Op {
        u32x4 a;
        f32x4 u, v;
        uint32_t nu, nv;
      };
      Walk w0(rd, c, 8 * b0 + 2 * j), w1(rd, c, 8 * b0 + 2 * j + 1);
      walk_blocks<AHEAD>(b0, b1, [&](int) { return Two{w0.next(), w1.next()}; }, [&](int b, const Two& f) {
        return Op{W.at(ct, b), f.u.quad(), f.v.quad(), f.u.site, f.v.site};
      }, [&](const Op& o) { mul16(o.a, kept<L>(o.u, o.nu), kept<L>(o.v, o.nv)); });
    } else if (TR && c.ck == 2) {
      // The last convolution's transpose, a tap's two products rounded together before they
      // are added: W_1 g_1, then W_0 g_0 + that by lane groups 0 and 1 of one MFMA per tap.
      struct Four {
        P at[4];
      };
      struct Op {
        u32x4 a;
        float v[4];
        uint32_t n[4];
      };
      const int e = 1 - (j & 1);
      walk_blocks<AHEAD>(b0, b1, [&](int b) {
        Four f;
#pragma unroll
        for (int r = 0; r < 4; ++r) f.at[r] = pair_at(rd, c, 2 * (4 * b + r) + e);
        return f;
      }, [&](int b, const Four& f) {
        Op o{W.at(ct, b), {}, {}};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          o.v[r] = *f.at[r].get();
          o.n[r] = f.at[r].site;
        }
        return o;
      }, [&](const Op& o) {
        f32x4 p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          p[r] = fused::mfma(__uint_as_float(o.a[r]), masked(kept<L>(o.v[r], o.n[r]), (j - 2) >> 31),
                             f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int r = 0; r < 4; ++r) s += p[r];
      });
    } else if (c.ck == 8) {
      // channels j and 4 + j of taps 2 b and 2 b + 1
      struct Two {
        P u, v;
      };
      struct Op {
        u32x4 a;
        f32x2 u, v;
        uint32_t nv;
      };
      using E = typename R::Entry;
      const float* p = rd.base + (j >> 1) * rd.ps + 2 * (j & 1);
      const int step = R::rev ? -rd.V : rd.V;
      const E* first = rd.nb + (R::rev ? rd.T - 1 : 0) * rd.V;
      walk_blocks<AHEAD>(b0, b1, [&](int b) {
        const E* row = first + 2 * b * step;
        return Two{{p, row[0]}, {p, row[step]}};
      }, [&](int b, const Two& f) { return Op{W.at(ct, b), f.u.pair(), f.v.pair(), f.v.site}; },
      [&](const Op& o) {  // (tap 2 b is never past the last)
        mul(o.a, f32x4{o.u[0], o.u[1], kept<L>(o.v[0], o.nv), kept<L>(o.v[1], o.nv)});
      });
    } else {
      struct Op {
        u32x4 a;
        f32x4 v;
        uint32_t n;
      };
      Walk w(rd, c, 4 * b0 + j);
      walk_blocks<AHEAD>(b0, b1, [&](int) { return w.next(); }, [&](int b, const P& f) {
        return Op{W.at(ct, b), f.quad(), f.site};
      }, [&](const Op& o) { mul(o.a, kept<L>(o.v, o.n)); });
    }
  }
  return s;
}

// Tree convolution without its bias.  SPLIT (in LDS): the sums part and part + 4 only, two
// scalars of a block's eight per lane.
template <bool SPLIT, class R>
__device__ __forceinline__ f32x4 tree(const R& rd, const ConvDir& c, const Weights& W, int ct, int j0, int part) {
  constexpr bool L = R::lds;
  constexpr int NS = SPLIT ? 2 : 8, AHEAD = L ? 0 : 2;
  f32x4 s[NS];
#pragma unroll
  for (int e = 0; e < NS; ++e) s[e] = f32x4{0.f, 0.f, 0.f, 0.f};
  struct A {
    float a[NS];
  };
  auto weights = [&](int b) {
    A o;
    if constexpr (SPLIT) {
      o.a[0] = W.elem(ct, 2 * b, part);
      o.a[1] = W.elem(ct, 2 * b + 1, part);
    } else {
      const u32x4 a0 = W.at(ct, 2 * b), a1 = W.at(ct, 2 * b + 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) o.a[e] = __uint_as_float(e < 4 ? a0[e & 3] : a1[e & 3]);
    }
    return o;
  };
  struct Sites {
    uint32_t n[NS];
  };
  struct Op {
    A w;
    float v[NS];
    Sites f;
  };
  auto mul = [&](const Op& o) {
#pragma unroll
    for (int e = 0; e < NS; ++e) s[e] = fused::mfma(o.w.a[e], kept<L>(o.v[e], o.f.n[e]), s[e]);
  };
  const int j = opaque(j0);
  auto pair = [&](int b, int e) { return 32 * b + 8 * j + (SPLIT ? part + 4 * e : e); };
  if constexpr (IsField<R>::value) {
    walk_blocks<AHEAD>(0, c.nb, [&](int b) {
      Sites f;
#pragma unroll
      for (int e = 0; e < NS; ++e) f.n[e] = rd.find(pair(b, e));
      return f;
    }, [&](int b, const Sites& f) {
      Op o{weights(b), {}, f};
#pragma unroll
      for (int e = 0; e < NS; ++e) o.v[e] = rd.get(f.n[e]);
      return o;
    }, mul);
  } else {
    using P = typename R::Place;
    if ((c.ck & 3) != 0) {
      struct Ats {
        P at[NS];
      };
      walk_blocks<AHEAD>(0, c.nb, [&](int b) {
        Ats f;
#pragma unroll
        for (int e = 0; e < NS; ++e) f.at[e] = pair_at(rd, c, pair(b, e));
        return f;
      }, [&](int b, const Ats& f) {
        Op o{weights(b), {}, {}};
#pragma unroll
        for (int e = 0; e < NS; ++e) {
          o.v[e] = *f.at[e].get();
          o.f.n[e] = f.at[e].site;
        }
        return o;
      }, mul);
    } else {
      struct Two {
        P u, v;
      };
      Walk w0(rd, c, 2 * j), w1(rd, c, 2 * j + 1);
      walk_blocks<AHEAD>(0, c.nb, [&](int) { return Two{w0.next(), w1.next()}; }, [&](int b, const Two& f) {
        Op o{weights(b), {}, {}};
        if constexpr (SPLIT) {
          o.v[0] = f.u.get()[part];
          o.v[1] = f.v.get()[part];
        } else {
          const f32x4 u0 = f.u.quad(), u1 = f.v.quad();
#pragma unroll
          for (int e = 0; e < 8; ++e) o.v[e] = e < 4 ? u0[e & 3] : u1[e & 3];
        }
#pragma unroll
        for (int e = 0; e < NS; ++e) o.f.n[e] = 2 * e < NS ? f.u.site : f.v.site;
        return o;
      }, mul);
    }
  }
  if constexpr (SPLIT) return s[0] + s[1];
  else return ((s[0] + s[4]) + (s[2] + s[6])) + ((s[1] + s[5]) + (s[3] + s[7]));
}

}  // namespace net
}  // namespace lfs
