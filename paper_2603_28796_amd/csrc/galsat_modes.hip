// Straight-through Gumbel training mode and the hand-off kernels
// (candidate pool, confidence, selection) for gfx950.
#include "galsat_device.h"

namespace galsat {

// ------------------------------------------- straight-through Gumbel mode
//
// Two logits per (variable, restart) go through a temperature softmax after
// Gumbel(0,1) noise (Section 3.2, Eq. 3); the forward uses the hard argmax
// (Eq. 4) and the backward the soft probabilities.  With two states only the
// logit difference d = theta1 - theta0 and the noise difference
// l = g1 - g0 matter: y1 = sigma((d + l) / tau), x_hat = [d + l > 0].

__global__ __launch_bounds__(256) void k_gumbel_noise(float* out, int32_t ldo, int32_t n, int32_t R,
                                                      uint64_t seed, int32_t t) {
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int r = blockIdx.y * 64 + lane;
  if (r >= R) return;
  for (int64_t v = (int64_t)blockIdx.x * 4 + w; v < n; v += (int64_t)gridDim.x * 4)
    out[v * ldo + r] = gumbel_diff(seed, t, v, r);
}

// Hard point of the step: xh = [d + l > 0] (FP32 sum; a tie goes to state
// 0), keeping l for the update.  noise: caller-given l or null to draw it.
__global__ __launch_bounds__(256) void k_gumbel_prep(const float* d, int32_t ldd, const float* noise,
                                                     int32_t ldn, uint64_t seed, int32_t t,
                                                     int32_t n, int32_t R, float* xh, float* nb,
                                                     int32_t ld) {
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int r = blockIdx.y * 64 + lane;
  if (r >= R) return;
  for (int64_t v = (int64_t)blockIdx.x * 4 + w; v < n; v += (int64_t)gridDim.x * 4) {
    const float l = noise ? noise[v * ldn + r] : gumbel_diff(seed, t, v, r);
    const float s = d[v * ldd + r] + l;
    xh[v * ld + r] = s > 0.0f ? 1.0f : 0.0f;
    nb[v * ld + r] = l;
  }
}

// Soft backward and update (gumbel_apply) from the float gradient G: the
// path of formulas whose counts the bit planes do not hold (galsat_hard.hip).
__global__ __launch_bounds__(256) void k_gumbel_update(float* d, int32_t ldd, const float* nb,
                                                       const float* G, int32_t ld, float* mom,
                                                       float* vel, int32_t ldm, int32_t n,
                                                       int32_t R, GumbelOpt o, int32_t adam) {
  const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int r = blockIdx.y * 64 + lane;
  if (r >= R) return;
  for (int64_t v = (int64_t)blockIdx.x * 4 + w; v < n; v += (int64_t)gridDim.x * 4) {
    float mo = adam ? mom[v * ldm + r] : 0.0f, ve = adam ? vel[v * ldm + r] : 0.0f;
    const float dv = d[v * ldd + r], l = nb[v * ld + r];
    const double G1 = (double)G[v * ld + r];
    d[v * ldd + r] = adam ? gumbel_apply<true>(dv, l, G1, o, mo, ve)
                          : gumbel_apply<false>(dv, l, G1, o, mo, ve);
    if (adam) {
      mom[v * ldm + r] = mo;
      vel[v * ldm + r] = ve;
    }
  }
}

// ---------------------------------------------------------- hand-off
//
// Candidate pool of Section 3.3.1, Eq. (8): candidate k of formula f adds
// the noise difference of "step" k, restart 0 to the logit difference of
// f's selected restart and takes the argmax; its confidence is the
// perturbed probability of the value taken.
// A thread takes one variable through a run of candidates, so the logit
// difference (a column of d, a line per variable) is read once per run and
// not once per candidate.  100 candidates of 100,000 variables at a stride
// of 64 restarts: 189 us with a thread per candidate and variable.
__global__ __launch_bounds__(256) void k_candidates(const float* __restrict__ d, int32_t ldd,
                                                    const int32_t* __restrict__ var_formula,
                                                    const int32_t* __restrict__ best, int32_t n,
                                                    int32_t num, int32_t run, uint64_t seed,
                                                    double inv_tau, uint8_t* __restrict__ assign,
                                                    float* __restrict__ conf) {
  const int k0 = blockIdx.y * run, k1 = min(num, k0 + run);
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    const int r = best[var_formula[v]];
    const float dv = d[v * ldd + r];
    for (int k = k0; k < k1; ++k) {
      const float l = gumbel_diff(seed, k, v, 0);
      // the probability of the value taken: the sigmoid of |d + l| / tau
      assign[(int64_t)k * n + v] = dv + l > 0.0f ? 1 : 0;
      conf[(int64_t)k * n + v] = (float)recip64(1.0 + exp_neg(((double)dv + (double)l) * inv_tau));
    }
  }
}

// Unperturbed confidence max(p, 1 - p), p = sigma(d / tau), of each
// variable at its formula's selected restart (Section 3.3.2).
__global__ __launch_bounds__(256) void k_confidence(const float* d, int32_t ldd,
                                                    const int32_t* var_formula, const int32_t* best,
                                                    int32_t n, double inv_tau, float* conf) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    conf[v] = (float)recip64(1.0 + exp_neg((double)d[v * ldd + best[var_formula[v]]] * inv_tau));
  }
}

// Selection of the S_f most (HIGH) or least confident variables of formula
// f in candidate k, ties to the lower index, written in increasing index
// order.  Keys are 64-bit: confidence bits (inverted for LOW) above the
// inverted local index, so every key is distinct and larger = preferred.
// One workgroup per (formula, candidate) narrows the range of keys that holds
// the S-th largest: 2,048 bins of equal width over the range (at first the
// span of the confidences, so keys that share their top digits are spread at
// once), a scan for the bin, the bin's range next, until all keys left in the
// range are selected.  As soon as few keys are at or above the range they are
// kept in LDS and the data are not read again.  At most kSelRank selected
// indices are put in order by counting the smaller ones, more by a
// compaction of the data in index order.
// What bounds it: the sweeps of the values by one workgroup (kSelU loads a
// thread in flight), so a long formula is cut into parts first
// (k_select_part).
template <bool HIGH>
__device__ __forceinline__ uint64_t sel_key(float c, int local) {
  const uint32_t b = __float_as_uint(c);
  const uint64_t hi = HIGH ? b : ~b;
  return (hi << 32) | (uint64_t)(~(uint32_t)local);
}

// Adds one to hist[bin] for every active lane, with one atomic when they all
// name the same bin.
__device__ __forceinline__ void hist_add(uint32_t* hist, bool act, uint32_t bin) {
  const uint64_t am = __ballot(act);
  if (am == 0) return;
  const int lead = __builtin_ctzll(am);
  const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)bin, lead);
  if (__ballot(act && bin == lb) == am) {
    if ((int)(threadIdx.x & 63) == lead) atomicAdd(&hist[lb], (uint32_t)__popcll(am));
  } else if (act) {
    atomicAdd(&hist[bin], 1u);
  }
}

constexpr int kSelU = 16;       // confidence loads in flight per thread
constexpr int kSelThreads = 1024;
constexpr int kSelBins = 2048;  // two per thread
constexpr int kSelList = 4096;  // keys kept in LDS
constexpr int kSelRank = 512;   // selected indices ordered by counting

constexpr int kSelPart = 8;     // values a thread of k_select_part holds

// fn(value, index, in range) for every element, whole waves in step
template <class T, class Fn>
__device__ __forceinline__ void sel_sweep(const T* c, int nf, Fn fn) {
  for (int base = 0; base < nf; base += kSelThreads * kSelU) {
    T cv[kSelU];
#pragma unroll
    for (int u = 0; u < kSelU; ++u) {
      const int i = base + u * kSelThreads + (int)threadIdx.x;
      cv[u] = i < nf ? c[i] : T(0);
    }
#pragma unroll
    for (int u = 0; u < kSelU; ++u) {
      const int i = base + u * kSelThreads + (int)threadIdx.x;
      if (base + u * kSelThreads < nf) fn(cv[u], i, i < nf);
    }
  }
}

// Position in a list for every active lane, the wave's lanes next to each other.
__device__ __forceinline__ int list_slot(int* count, bool act) {
  const uint64_t m = __ballot(act);
  if (m == 0) return 0;
  const int lane = threadIdx.x & 63, lead = __builtin_ctzll(m);
  int at = 0;
  if (lane == lead) at = atomicAdd(count, __popcll(m));
  at = __builtin_amdgcn_readlane(at, lead);
  return at + __popcll(m & ((1ULL << lane) - 1ULL));
}

struct SelShared {
  uint32_t hist[kSelBins];
  uint32_t min, max, bin, rank, cnt;
  int count;
  int wave_tot[kSelThreads / 64];
};

// The S-th largest key (S of them are >= it).  sweep(fn) calls fn(key, valid)
// for every key, whole waves in step; after(lo, above) follows every level
// that does not end it: `above` keys are >= lo.
template <class Sweep, class After>
__device__ __forceinline__ uint64_t sel_threshold(SelShared& sh, int S, Sweep sweep, After after) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) {
    sh.min = 0xffffffffu;
    sh.max = 0;
    sh.count = 0;
  }
  __syncthreads();
  {
    uint32_t mn = 0xffffffffu, mx = 0;
    sweep([&](uint64_t key, bool in) {
      const uint32_t b = (uint32_t)(key >> 32);
      mn = in && b < mn ? b : mn;
      mx = in && b > mx ? b : mx;
    });
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t a = (uint32_t)__shfl_xor((int)mn, d, 64), b = (uint32_t)__shfl_xor((int)mx, d, 64);
      mn = a < mn ? a : mn;
      mx = b > mx ? b : mx;
    }
    if (lane == 0) {
      atomicMin(&sh.min, mn);
      atomicMax(&sh.max, mx);
    }
  }
  __syncthreads();
  // keys of [lo, hi] hold the rank-th largest from the top of the range, all
  // keys above hi are selected
  uint64_t lo = (uint64_t)sh.min << 32, hi = (uint64_t)sh.max << 32 | 0xffffffffULL;
  int rank = S;
  // a range of 64 bits is one key after six levels
  for (int level = 0; level < 8; ++level) {
    const uint64_t span = hi - lo;
    const int width = span ? 64 - __clzll((long long)span) : 0;
    const int shift = width > 11 ? width - 11 : 0;  // span >> shift < kSelBins
    sh.hist[tid] = 0;
    sh.hist[tid + kSelThreads] = 0;
    __syncthreads();
    sweep([&](uint64_t key, bool in) {
      hist_add(sh.hist, in && key >= lo && key <= hi,
               (uint32_t)((key - lo) >> shift) & (kSelBins - 1));
    });
    __syncthreads();
    // thread t has the bins 2047 - 2t and 2046 - 2t
    const int b1 = kSelBins - 1 - 2 * tid;
    const int h1 = (int)sh.hist[b1], h0 = (int)sh.hist[b1 - 1];
    int incl = h1 + h0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(incl, d, 64);
      if (lane >= d) incl += y;
    }
    if (lane == 63) sh.wave_tot[w] = incl;
    __syncthreads();
    for (int u = 0; u < w; ++u) incl += sh.wave_tot[u];
    const int before = incl - h1 - h0;
    if (before < rank && rank <= incl) {
      const bool second = before + h1 < rank;
      sh.bin = (uint32_t)(second ? b1 - 1 : b1);
      sh.rank = (uint32_t)(rank - before - (second ? h1 : 0));
      sh.cnt = (uint32_t)(second ? h0 : h1);
    }
    __syncthreads();
    lo += (uint64_t)sh.bin << shift;
    const uint64_t wide = ((uint64_t)1 << shift) - 1;  // compared as widths: lo + wide can pass 2^64
    hi = hi - lo < wide ? hi : lo + wide;
    rank = (int)sh.rank;
    const int cnt = (int)sh.cnt;
    if (cnt == rank) break;
    after(lo, S - rank + cnt);
  }
  return lo;
}

// KEYS: the candidate's keys come from k_select_part (`keys`, nk of them a
// candidate, 0: none) instead of the confidences; one formula then.
template <bool HIGH, bool KEYS>
__global__ __launch_bounds__(kSelThreads) void k_select(const float* __restrict__ conf, int32_t n,
                                                        const uint64_t* __restrict__ keys, int32_t nk,
                                                        const int32_t* __restrict__ f_vbeg,
                                                        const int32_t* __restrict__ sel_off,
                                                        int32_t stot, int32_t* __restrict__ out) {
  constexpr int W = kSelThreads / 64;
  const int f = blockIdx.x, k = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int v0 = f_vbeg[f], nf = f_vbeg[f + 1] - v0;
  // one formula: its selections are all of them
  const int so = sel_off ? sel_off[f] : 0;
  const int S = sel_off ? sel_off[f + 1] - so : stot;
  if (S <= 0) return;
  const float* c = conf + (int64_t)k * n + v0;
  int32_t* o = out + (int64_t)k * stot + so;
  __shared__ SelShared sh;
  __shared__ uint64_t list[kSelList];
  __shared__ uint32_t sel[kSelRank];
  __shared__ int s_list;
  if (tid == 0) s_list = 0;
  bool listed = false;
  auto sweep = [&](auto fn) {
    if (listed) {
      const int ln = s_list;
      for (int b = 0; b < ln; b += kSelThreads) {
        const bool in = b + tid < ln;
        fn(in ? list[b + tid] : 0, in);
      }
    } else if constexpr (KEYS) {
      sel_sweep(keys + (int64_t)k * nk, nk, [&](uint64_t key, int, bool in) { fn(key, in && key != 0); });
    } else {
      sel_sweep(c, nf, [&](float x, int i, bool in) { fn(sel_key<HIGH>(x, i), in); });
    }
  };
  const uint64_t lo = sel_threshold(sh, S, sweep, [&](uint64_t from, int above) {
    if (listed || S > kSelRank || above > kSelList) return;
    sweep([&](uint64_t key, bool in) {
      const bool keep = in && key >= from;
      const int at = list_slot(&s_list, keep);
      if (keep) list[at] = key;
    });
    listed = true;
    __syncthreads();
  });
  // keys >= lo are the selection
  if (KEYS || S <= kSelRank) {
    sweep([&](uint64_t key, bool in) {
      const bool keep = in && key >= lo;
      const int at = list_slot(&sh.count, keep);
      if (keep) sel[at] = ~(uint32_t)key;
    });
    __syncthreads();
    if (tid < S) {
      const uint32_t mine = sel[tid];
      int less = 0;
      for (int j = 0; j < S; ++j) less += sel[j] < mine ? 1 : 0;
      o[less] = v0 + (int)mine;
    }
    return;
  }
  // each wave a contiguous run of whole 64s: counts, then their prefix, then
  // the indices in order
  const int per = ((nf + W - 1) / W + 63) / 64 * 64;
  const int i0 = w * per, i1 = min(nf, i0 + per);
  int mine = 0;
  for (int i = i0 + lane; i - lane < i1; i += 64)
    mine += __popcll(__ballot(i < i1 && sel_key<HIGH>(i < i1 ? c[i] : 0.0f, i) >= lo));
  __syncthreads();
  if (lane == 0) sh.wave_tot[w] = mine;
  __syncthreads();
  int pos = 0;
  for (int u = 0; u < w; ++u) pos += sh.wave_tot[u];
  for (int i = i0 + lane; i - lane < i1; i += 64) {
    const bool keep = i < i1 && sel_key<HIGH>(i < i1 ? c[i] : 0.0f, i) >= lo;
    const uint64_t m = __ballot(keep);
    if (keep) o[pos + __popcll(m & ((1ULL << lane) - 1ULL))] = v0 + i;
    pos += __popcll(m);
  }
}

// First stage of a selection from one long formula: a workgroup holds one
// part of the confidences in registers, finds the part's own S largest and
// writes their keys (0 for the rest when the part has fewer values); the
// selection is among them.  One workgroup a candidate left the chip to its
// sweeps: the 7 least confident of 100,000 took 85 us, the 50 most confident
// of 100 candidates 107 us.
template <bool HIGH>
__global__ __launch_bounds__(kSelThreads) void k_select_part(const float* __restrict__ conf, int32_t n,
                                                             int32_t S, uint64_t* __restrict__ keys,
                                                             int32_t nk) {
  const int tid = threadIdx.x, k = blockIdx.y;
  const int base = blockIdx.x * (kSelThreads * kSelPart);
  const float* c = conf + (int64_t)k * n;
  uint64_t* o = keys + (int64_t)k * nk + (int64_t)blockIdx.x * S;
  __shared__ SelShared sh;
  float cv[kSelPart];
#pragma unroll
  for (int u = 0; u < kSelPart; ++u) {
    const int i = base + u * kSelThreads + tid;
    cv[u] = i < n ? c[i] : 0.0f;
  }
  auto sweep = [&](auto fn) {
#pragma unroll
    for (int u = 0; u < kSelPart; ++u) {
      const int i = base + u * kSelThreads + tid;
      if (base + u * kSelThreads < n) fn(sel_key<HIGH>(cv[u], i), i < n);
    }
  };
  const int have = min(n - base, kSelThreads * kSelPart);
  uint64_t lo = 0;
  if (have > S) {
    lo = sel_threshold(sh, S, sweep, [](uint64_t, int) {});
  } else {
    if (tid == 0) sh.count = 0;
    __syncthreads();
  }
  sweep([&](uint64_t key, bool in) {
    const bool keep = in && key >= lo;
    const int at = list_slot(&sh.count, keep);
    if (keep) o[at] = key;
  });
  for (int i = have + tid; i < S; i += kSelThreads) o[i] = 0;
}

// Offsets of a selection: formula f takes min(n_f, max(min_count,
// ceil(frac n_f))) variables, as the host counts them.  One workgroup.
__global__ __launch_bounds__(1024) void k_sel_offsets(const int32_t* f_vbeg, int32_t F, float frac,
                                                      int32_t min_count, int32_t* off) {
  __shared__ int wave_tot[16], s_run;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) {
    s_run = 0;
    off[0] = 0;
  }
  __syncthreads();
  for (int base = 0; base < F; base += 1024) {
    const int f = base + tid;
    int cnt = 0;
    if (f < F) {
      const int nf = f_vbeg[f + 1] - f_vbeg[f];
      int64_t c = (int64_t)ceil((double)frac * (double)nf);
      c = c < min_count ? min_count : c;
      cnt = (int)(c < nf ? c : nf);
    }
    int incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(incl, d, 64);
      if (lane >= d) incl += y;
    }
    if (lane == 63) wave_tot[w] = incl;
    __syncthreads();
    for (int u = 0; u < w; ++u) incl += wave_tot[u];
    incl += s_run;
    if (f < F) off[f + 1] = incl;
    __syncthreads();
    if (tid == 1023) s_run = incl;
    __syncthreads();
  }
}

// ------------------------------------------------------------ launchers

hipError_t launch_gumbel_noise(float* out, int32_t ldo, int32_t n, int32_t R, uint64_t seed,
                               int32_t t, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  dim3 grid(grid_x_for(((int64_t)n + 3) / 4), (R + 63) / 64), block(256);
  hipLaunchKernelGGL(k_gumbel_noise, grid, block, 0, s, out, ldo, n, R, seed, t);
  return hipGetLastError();
}

hipError_t launch_gumbel_prep(const float* d, int32_t ldd, const float* noise, int32_t ldn,
                              uint64_t seed, int32_t t, int32_t n, int32_t R, float* xh, float* nb,
                              int32_t ld, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  dim3 grid(grid_x_for(((int64_t)n + 3) / 4), (R + 63) / 64), block(256);
  hipLaunchKernelGGL(k_gumbel_prep, grid, block, 0, s, d, ldd, noise, ldn, seed, t, n, R, xh, nb, ld);
  return hipGetLastError();
}

hipError_t launch_gumbel_update(float* d, int32_t ldd, const float* nb, const float* G, int32_t ld,
                                float* mom, float* vel, int32_t ldm, int32_t n, int32_t R,
                                const GumbelOpt& o, int32_t adam, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  dim3 grid(grid_x_for(((int64_t)n + 3) / 4), (R + 63) / 64), block(256);
  hipLaunchKernelGGL(k_gumbel_update, grid, block, 0, s, d, ldd, nb, G, ld, mom, vel, ldm, n, R, o,
                     adam);
  return hipGetLastError();
}

hipError_t launch_candidates(const float* d, int32_t ldd, const int32_t* var_formula,
                             const int32_t* best, int32_t n, int32_t num, uint64_t seed, float tau,
                             uint8_t* assign, float* conf, hipStream_t s) {
  if (n <= 0 || num <= 0) return hipSuccess;
  // runs of candidates as long as about 4,096 workgroups remain
  const int64_t gx = grid_x_for(((int64_t)n + 255) / 256);
  int run = (int)std::min<int64_t>(std::max<int64_t>(1, gx * num / 4096), num);
  run = std::max(run, (num + 65534) / 65535);
  dim3 grid((uint32_t)gx, (num + run - 1) / run), block(256);
  hipLaunchKernelGGL(k_candidates, grid, block, 0, s, d, ldd, var_formula, best, n, num, run, seed,
                     1.0 / (double)tau, assign, conf);
  return hipGetLastError();
}

hipError_t launch_confidence(const float* d, int32_t ldd, const int32_t* var_formula,
                             const int32_t* best, int32_t n, float tau, float* conf, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_confidence, dim3(grid_x_for(((int64_t)n + 255) / 256)), dim3(256), 0, s, d,
                     ldd, var_formula, best, n, 1.0 / (double)tau, conf);
  return hipGetLastError();
}

hipError_t launch_sel_offsets(const int32_t* f_vbeg, int32_t F, float frac, int32_t min_count,
                              int32_t* off, hipStream_t s) {
  hipLaunchKernelGGL(k_sel_offsets, dim3(1), dim3(1024), 0, s, f_vbeg, F, frac, min_count, off);
  return hipGetLastError();
}

// Keys of the first stage for one formula, 0: not worth it (one sweep of a
// workgroup, an ordering by compaction, or nearly all values are kept).
int64_t select_part_keys(int32_t n, int64_t S) {
  const int64_t part = kSelThreads * kSelPart, parts = (n + part - 1) / part;
  return parts > 1 && S <= kSelRank && parts * S * 4 <= n ? parts * S : 0;
}

namespace {

template <bool HIGH>
hipError_t select_go(const float* conf, int32_t n, int32_t F, const int32_t* f_vbeg,
                     const int32_t* sel_off, int32_t stot, int32_t num, uint64_t* keys, int32_t* out,
                     hipStream_t s) {
  const dim3 grid(F, num), block(kSelThreads);
  if (!keys) {
    hipLaunchKernelGGL((k_select<HIGH, false>), grid, block, 0, s, conf, n, (const uint64_t*)nullptr, 0,
                       f_vbeg, sel_off, stot, out);
    return hipGetLastError();
  }
  const int32_t nk = (int32_t)select_part_keys(n, stot);
  hipLaunchKernelGGL((k_select_part<HIGH>), dim3(nk / stot, num), block, 0, s, conf, n, stot, keys, nk);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_select<HIGH, true>), grid, block, 0, s, conf, n, keys, nk, f_vbeg, sel_off, stot,
                     out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const float* conf, int32_t n, int32_t F, const int32_t* f_vbeg,
                         const int32_t* sel_off, int32_t stot, int32_t num, bool highest,
                         uint64_t* keys, int32_t* out, hipStream_t s) {
  if (F <= 0 || num <= 0 || stot <= 0) return hipSuccess;
  return highest ? select_go<true>(conf, n, F, f_vbeg, sel_off, stot, num, keys, out, s)
                 : select_go<false>(conf, n, F, f_vbeg, sel_off, stot, num, keys, out, s);
}

}  // namespace galsat
