// Independence Metropolis-Hastings chains (paper Sec. 1, the MH test that
// corrects flow proposals to exp(-S)/Z) and the FP64 HMC baseline (paper
// Sec. 2.2, HMC for the same theory, "to compare results").
#include "lfs_common.hpp"

namespace lfs {
namespace {

// Decision i of a chain whose current log-weight is w_cur: log u_i < w_i - w_cur, one
// rounded FP64 subtraction and one comparison, made here for 64 proposals at a time, one
// per lane.  A chain is sequential only through w_cur, which changes when a proposal is
// accepted, so a chunk's decisions follow from its accepted positions: the first one
// after the entry, then from each accepted position the next one.
__device__ __forceinline__ uint64_t read_lane(uint64_t v, int l) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32;
}
__device__ __forceinline__ double read_lane(double v, int l) {
  return __longlong_as_double((long long)read_lane((uint64_t)__double_as_longlong(v), l));
}

// The chunk's results from the bit mask of its accepted positions (g0: the number of its
// first proposal): cur_idx and accepted of this lane's proposal.
__device__ __forceinline__ void put_chunk(uint64_t path, int lane, bool valid, int64_t g0, int64_t idx_cur,
                                          int64_t* cur_idx, uint8_t* accepted) {
  const uint64_t upto = path & (~0ull >> (63 - lane));
  if (!valid) return;
  *cur_idx = upto ? g0 + (63 - __builtin_clzll(upto)) : idx_cur;
  if (accepted) *accepted = (uint8_t)((path >> lane) & 1);
}

// One wave per chain: every accepted proposal costs one test of the chunk against the new
// w_cur (about 70 cycles), every chunk one more; the next chunk is loaded meanwhile.  64
// proposals: 6.4 -> 1.8 us against one lane testing proposal after proposal.
// Chain c reads proposals [offsets[c], offsets[c+1]) (rectangular calls pass
// offsets == NULL and use [c * n_prop, (c+1) * n_prop)); its state lives at
// state[state_index[c]] (or state[c]).
// Positions are unsigned: the chunk after the last one is looked up, which for the longest
// chain (2^31 - 1 proposals) is past the largest int.
__global__ void __launch_bounds__(64) k_mh_chain(int n_prop_rect, const int64_t* __restrict__ offsets,
                                                 const double* __restrict__ logw,
                                                 const double* __restrict__ log_u,
                                                 lfs_chain_state* __restrict__ states,
                                                 const int32_t* __restrict__ state_index,
                                                 int64_t* __restrict__ cur_idx,
                                                 uint8_t* __restrict__ accepted) {
  const int c = blockIdx.x, lane = threadIdx.x;
  const size_t base = offsets ? (size_t)offsets[c] : (size_t)c * n_prop_rect;
  const int count = offsets ? (int)(offsets[c + 1] - offsets[c]) : n_prop_rect;
  const unsigned n_prop = (unsigned)max(count, 0);
  lfs_chain_state* state = states + (state_index ? state_index[c] : c);
  lfs_chain_state st = *state;
  const int64_t seen0 = st.n_seen;
  // lanes past the end never accept
  auto load = [&](unsigned k, double& w, double& u) {
    w = k < n_prop ? logw[base + k] : 0.0;
    u = k < n_prop ? log_u[base + k] : HUGE_VAL;
  };
  double w, u, wn, un;
  load(lane, w, u);
  for (unsigned k0 = 0; k0 < n_prop; k0 += kWave) {
    load(k0 + kWave + lane, wn, un);
    const int64_t g0 = seen0 + k0;
    uint64_t path = 0, open = ~0ull;  // open: positions after the last accepted one
    if (!st.has_state) {
      st.has_state = 1;
      st.w_cur = read_lane(w, 0);
      path = 1;
      open = ~1ull;
    }
    const uint64_t seed = path;
    for (;;) {
      const uint64_t m = __ballot(u < w - st.w_cur) & open;
      if (m == 0) break;
      const int e = __builtin_ctzll(m);
      path |= 1ull << e;
      open = e == 63 ? 0 : ~0ull << (e + 1);
      st.w_cur = read_lane(w, e);
    }
    const int64_t before = st.idx_cur;
    if (path) st.idx_cur = g0 + (63 - __builtin_clzll(path));
    st.n_acc += __builtin_popcountll(path & ~seed);
    const unsigned k = k0 + lane;
    put_chunk(path, lane, k < n_prop, g0, before, cur_idx + base + k, accepted ? accepted + base + k : nullptr);
    w = wn;
    u = un;
  }
  if (lane == 0) {
    st.n_seen = seen0 + count;
    *state = st;
  }
}

// Long chains in two launches.  Whether proposal i of a chunk would be accepted from
// proposal k < i as the current state depends on neither the chain's past nor other
// chunks, so every chunk's 64 rows are tested in parallel (64 subtractions, comparisons
// and ballots of one wave), giving each position's next accepted one; pointer doubling
// (six rounds) turns that into the mask of all positions accepted after it, itself
// included.  The masks wait in cur_idx, 8 bytes per proposal.  The second launch walks the
// chunks in order: one test against w_cur finds the first accepted position, its mask the
// rest.  65536 proposals at acceptance 0.43: 5046 -> 198 us, of which the walk 192
// (2.9 ns per proposal; lane 0 alone took 77).
__global__ void __launch_bounds__(256) k_mh_paths(int n_prop, const double* __restrict__ logw,
                                                  const double* __restrict__ log_u, int64_t* __restrict__ cur_idx) {
  const int lane = threadIdx.x & 63, k0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kWave;
  if (k0 >= n_prop) return;
  const size_t at = (size_t)blockIdx.y * n_prop + k0 + lane;
  const bool valid = k0 + lane < n_prop;
  const double w = valid ? logw[at] : 0.0, u = valid ? log_u[at] : HUGE_VAL;
  int next = 0;
#pragma unroll
  for (int k = 0; k < kWave; ++k) {
    const uint64_t m = __ballot(u < w - read_lane(w, k)) & (k == 63 ? 0ull : ~0ull << (k + 1));
    next = lane == k ? (m ? __builtin_ctzll(m) : k) : next;
  }
  uint32_t lo = lane < 32 ? 1u << lane : 0u, hi = lane < 32 ? 0u : 1u << (lane - 32);
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    lo |= (uint32_t)__shfl((int)lo, next, kWave);
    hi |= (uint32_t)__shfl((int)hi, next, kWave);
    next = __shfl(next, next, kWave);
  }
  if (valid) cur_idx[at] = (int64_t)((uint64_t)hi << 32 | lo);
}

// The walk: wave 0 makes the decisions of a group of chunks from LDS (per chunk a
// subtraction, a comparison and a handful of scalar steps, all in one dependent chain)
// while the other three waves fetch the next group and write the results of the previous
// one, which as per-lane 64-bit arithmetic costs as much as the decisions (one wave doing
// both: 380 us).
constexpr int kWalkChunks = 16;  // chunks per group
// Longer chains take the other kernel: a group more than they have would be counted in int.
constexpr int kWalkMost = INT32_MAX - kWalkChunks * kWave;
__global__ void __launch_bounds__(256) k_mh_walk(int n_prop, const double* __restrict__ logw,
                                                 const double* __restrict__ log_u, lfs_chain_state* __restrict__ states,
                                                 int64_t* cur_idx, uint8_t* __restrict__ accepted) {
  constexpr int GP = kWalkChunks * kWave;
  __shared__ double sw[2][GP], su[2][GP];
  __shared__ uint64_t sp[2][GP], spath[2][kWalkChunks];
  __shared__ int64_t sbefore[2][kWalkChunks];
  const int c = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const size_t base = (size_t)c * n_prop;
  lfs_chain_state st = states[c];
  const int64_t seen0 = st.n_seen;
  const int groups = (n_prop + GP - 1) / GP;
  auto fetch = [&](int g, int first, int waves) {
    constexpr int MX = (kWalkChunks + 2) / 3;
    double w[MX], u[MX];
    uint64_t p[MX];
#pragma unroll
    for (int i = 0; i < MX; ++i) {
      const int ch = first + i * waves, k = g * GP + ch * kWave + lane;
      const bool ok = ch < kWalkChunks && k < n_prop;
      w[i] = ok ? logw[base + k] : 0.0;
      u[i] = ok ? log_u[base + k] : HUGE_VAL;  // lanes past the end never accept
      p[i] = ok ? (uint64_t)cur_idx[base + k] : 0ull;
    }
#pragma unroll
    for (int i = 0; i < MX; ++i) {
      const int ch = first + i * waves, o = ch * kWave + lane;
      if (ch < kWalkChunks) sw[g & 1][o] = w[i], su[g & 1][o] = u[i], sp[g & 1][o] = p[i];
    }
  };
  fetch(0, wv, 4);
  __syncthreads();
  for (int g = 0; g <= groups; ++g) {
    if (wv == 0) {
      if (g < groups) {
        const double *w = sw[g & 1], *u = su[g & 1];
        const uint64_t* p = sp[g & 1];
        double wl = w[lane], ul = u[lane];
        uint64_t pl = p[lane];
        const int chunks = min(kWalkChunks, (n_prop - g * GP + kWave - 1) / kWave);
        for (int i = 0; i < chunks; ++i) {
          const int nx = min(i + 1, kWalkChunks - 1) * kWave + lane;
          const double wn = w[nx], un = u[nx];
          const uint64_t pn = p[nx];
          uint64_t path = 0;
          const int64_t before = st.idx_cur;
          const uint64_t m = st.has_state ? __ballot(ul < wl - st.w_cur) : 1ull;
          if (m) {
            path = read_lane(pl, __builtin_ctzll(m));
            const int last = 63 - __builtin_clzll(path);
            st.w_cur = read_lane(wl, last);
            st.idx_cur = seen0 + (int64_t)g * GP + i * kWave + last;
            st.n_acc += __builtin_popcountll(path) - (st.has_state ? 0 : 1);
            st.has_state = 1;
          }
          if (lane == 0) spath[g & 1][i] = path, sbefore[g & 1][i] = before;
          wl = wn;
          ul = un;
          pl = pn;
        }
      }
    } else {
      if (g > 0) {
        for (int i = wv - 1; i < kWalkChunks; i += 3) {
          const int kc = (g - 1) * GP + i * kWave, k = kc + lane;
          if (kc < n_prop)
            put_chunk(spath[(g - 1) & 1][i], lane, k < n_prop, seen0 + kc, sbefore[(g - 1) & 1][i], cur_idx + base + k,
                      accepted ? accepted + base + k : nullptr);
        }
      }
      if (g + 1 < groups) fetch(g + 1, wv - 1, 3);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    st.n_seen = seen0 + n_prop;
    states[c] = st;
  }
}

// Per-site action density and force from an LDS-resident FP64 field.  L is the
// compile-time LT where LT > 0 (a power of two: the coordinate arithmetic is shifts
// and masks), else the runtime value.
template <int DIM, int LT>
__device__ __forceinline__ void site_terms(const double* f, int n, int Lrt, double m2, double lam,
                                           double& dens, double& frc) {
  const int L = LT > 0 ? LT : Lrt;
  const double p = f[n];
  double nb = 0.0;
  int stride = 1;
#pragma unroll
  for (int mu = DIM - 1; mu >= 0; --mu) {
    const int c = (n / stride) % L;
    const int up = (c == L - 1) ? n - (L - 1) * stride : n + stride;
    const int dn = (c == 0) ? n + (L - 1) * stride : n - stride;
    nb += f[up] + f[dn];
    stride *= L;
  }
  const double lap = nb - 2.0 * DIM * p;
  const double p2 = p * p;
  dens = -p * lap + m2 * p2 + lam * p2 * p2;
  frc = -2.0 * lap + 2.0 * m2 * p + 4.0 * lam * p2 * p;
}

// One block per chain; phi, pi and the force stay in LDS for the whole
// trajectory.  Kick-drift-kick: the closing half-kick of a step and the opening
// half-kick of the next use the force at the same field, so it is evaluated
// once per step (and once at the start); both half-kicks are still applied as
// two separate subtractions, as the definition has them.  The last force pass
// also sums the final Hamiltonian.  Every thread owns sites tid, tid + blockDim, ...
// in every pass, so its kicks read only its own force entries.
template <int DIM, int LT>
__global__ void __launch_bounds__(256) k_hmc(int Lrt, double* __restrict__ phi,
                                             const double* __restrict__ pi0,
                                             const double* __restrict__ log_u,
                                             const double* __restrict__ m2p,
                                             const double* __restrict__ lamp, int per_sample,
                                             int n_steps, double dt, double* __restrict__ dH,
                                             uint8_t* __restrict__ accepted) {
  extern __shared__ double smem[];
  __shared__ double sh[16];
  const int L = LT > 0 ? LT : Lrt;
  int V = L;
  for (int i = 1; i < DIM; ++i) V *= L;
  double* f = smem;
  double* p = smem + V;
  double* F = smem + 2 * V;
  const int b = blockIdx.x;
  const double m2 = m2p[per_sample ? b : 0], lam = lamp[per_sample ? b : 0];
  for (int n = threadIdx.x; n < V; n += blockDim.x) {
    f[n] = phi[(size_t)b * V + n];
    p[n] = pi0[(size_t)b * V + n];
  }
  __syncthreads();
  double h = 0.0, dens, frc;
  for (int n = threadIdx.x; n < V; n += blockDim.x) {
    site_terms<DIM, LT>(f, n, L, m2, lam, dens, frc);
    F[n] = frc;
    h += 0.5 * p[n] * p[n] + dens;
  }
  const double H0 = block_sum(h, sh);  // ends with a barrier
  const double hdt = 0.5 * dt;
  h = 0.0;
  for (int s = 0; s < n_steps; ++s) {
    for (int n = threadIdx.x; n < V; n += blockDim.x) {
      p[n] = p[n] - hdt * F[n];
      f[n] = f[n] + dt * p[n];
    }
    __syncthreads();
    const bool last = s == n_steps - 1;
    for (int n = threadIdx.x; n < V; n += blockDim.x) {
      site_terms<DIM, LT>(f, n, L, m2, lam, dens, frc);
      F[n] = frc;
      p[n] = p[n] - hdt * frc;
      if (last) h += 0.5 * p[n] * p[n] + dens;
    }
    __syncthreads();  // the next drift rewrites f, which this pass read at neighbours
  }
  const double H1 = n_steps > 0 ? block_sum(h, sh) : H0;
  const double d = H1 - H0;
  const bool acc = log_u[b] < -d;
  if (acc)
    for (int n = threadIdx.x; n < V; n += blockDim.x) phi[(size_t)b * V + n] = f[n];
  if (threadIdx.x == 0) {
    dH[b] = d;
    accepted[b] = acc ? 1 : 0;
  }
}

__global__ void k_adam(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2,
                       float eps, float inv_bc1, float inv_bc2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] = p[i] - lr * (mi * inv_bc1) / (sqrtf(vi * inv_bc2) + eps);
  }
}

}  // namespace
}  // namespace lfs

extern "C" int32_t lfs_mh_chain(int32_t n_chains, int32_t n_prop, const double* logw,
                                const double* log_u, lfs_chain_state* state, int64_t* cur_idx,
                                uint8_t* accepted, void* stream) {
  LFS_RETURN_IF(n_chains < 0 || n_prop < 0, LFS_EINVAL);
  if (n_chains == 0 || n_prop == 0) return LFS_OK;
  LFS_RETURN_IF(!logw || !log_u || !state || !cur_idx, LFS_EINVAL);
  hipStream_t st = (hipStream_t)stream;
  // two launches take 12.5 us at 512 proposals whatever is accepted; one takes 9 to 16 us at
  // 256 (acceptance 0 to 0.85) and 13 to 30 at 512
  if (n_prop < 512 || n_chains > 65535 || n_prop > lfs::kWalkMost) {
    hipLaunchKernelGGL(lfs::k_mh_chain, dim3(n_chains), dim3(lfs::kWave), 0, st, n_prop, nullptr, logw, log_u, state,
                       nullptr, cur_idx, accepted);
    return lfs::launch_status();
  }
  const unsigned chunks = ((unsigned)n_prop + lfs::kWave - 1) / lfs::kWave;
  hipLaunchKernelGGL(lfs::k_mh_paths, dim3((chunks + 3) / 4, n_chains), dim3(256), 0, st, n_prop, logw, log_u, cur_idx);
  hipLaunchKernelGGL(lfs::k_mh_walk, dim3(n_chains), dim3(256), 0, st, n_prop, logw, log_u, state, cur_idx,
                     accepted);
  return lfs::launch_status();
}

extern "C" int32_t lfs_mh_chain_ragged(int32_t n_chains, const int64_t* offsets, const double* logw,
                                       const double* log_u, lfs_chain_state* states,
                                       const int32_t* state_index, int64_t* cur_idx,
                                       uint8_t* accepted, void* stream) {
  LFS_RETURN_IF(n_chains < 0, LFS_EINVAL);
  if (n_chains == 0) return LFS_OK;
  LFS_RETURN_IF(!offsets || !logw || !log_u || !states || !state_index || !cur_idx, LFS_EINVAL);
  hipLaunchKernelGGL(lfs::k_mh_chain, dim3(n_chains), dim3(lfs::kWave), 0, (hipStream_t)stream, 0,
                     offsets, logw, log_u, states, state_index, cur_idx, accepted);
  return lfs::launch_status();
}

extern "C" int32_t lfs_hmc_step(int32_t dim, int32_t L, int32_t B, double* phi, const double* pi0,
                                const double* log_u, const double* m2, const double* lam,
                                int32_t per_sample, int32_t n_steps, double dt, double* dH,
                                uint8_t* accepted, void* stream) {
  LFS_RETURN_IF(dim != 2 && dim != 3, LFS_EINVAL);
  LFS_RETURN_IF(L < 2 || B < 0 || n_steps < 0, LFS_EINVAL);
  const long V = dim == 2 ? (long)L * L : (long)L * L * L;
  LFS_RETURN_IF(V > 4096, LFS_EUNSUPPORTED);  // phi, pi and the force in at most 96 KB of LDS
  if (B == 0) return LFS_OK;
  LFS_RETURN_IF(!phi || !pi0 || !log_u || !m2 || !lam || !dH || !accepted, LFS_EINVAL);
  const size_t shm = 3 * (size_t)V * sizeof(double);
  hipStream_t st = (hipStream_t)stream;
  // compile-time lattice sizes for the common powers of two, the runtime L otherwise
  using Kern = void (*)(int, double*, const double*, const double*, const double*, const double*, int, int,
                        double, double*, uint8_t*);
  const int li = L == 4 ? 1 : L == 8 ? 2 : L == 16 ? 3 : 0;
  static const Kern k2[4] = {lfs::k_hmc<2, 0>, lfs::k_hmc<2, 4>, lfs::k_hmc<2, 8>, lfs::k_hmc<2, 16>};
  static const Kern k3[4] = {lfs::k_hmc<3, 0>, lfs::k_hmc<3, 4>, lfs::k_hmc<3, 8>, lfs::k_hmc<3, 16>};
  const Kern k = dim == 2 ? k2[li] : k3[li];
  if (shm > 64 * 1024)
    LFS_RETURN_IF(hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)shm) != hipSuccess,
                  LFS_EDEVICE);
  hipLaunchKernelGGL(k, dim3(B), dim3(256), shm, st, L, phi, pi0, log_u, m2, lam, per_sample, n_steps, dt, dH,
                     accepted);
  return lfs::launch_status();
}

extern "C" int32_t lfs_adam_step(int64_t n, float* p, const float* g, float* m, float* v, float lr,
                                 float b1, float b2, float eps, int64_t t, void* stream) {
  LFS_RETURN_IF(n <= 0 || t < 1 || !p || !g || !m || !v, LFS_EINVAL);
  const double bc1 = 1.0 - pow((double)b1, (double)t), bc2 = 1.0 - pow((double)b2, (double)t);
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(lfs::k_adam, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, n, p,
                     g, m, v, lr, b1, b2, eps, (float)(1.0 / bc1), (float)(1.0 / bc2));
  return lfs::launch_status();
}
