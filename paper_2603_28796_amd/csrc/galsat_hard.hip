// Straight-through Gumbel step on bit planes (gfx950).
//
// The forward of a step is at the hard point x_hat in {0, 1} (Section 3.2,
// Eq. 3-4), where every clause value U_t and every literal's partial product
// is 0 or 1: a literal's factor is one bit, the product of a clause's other
// factors is an AND, the gradient of a variable is the number of its negated
// occurrences whose other literals are all false minus that of its positive
// ones, and loss' is the unsat count.  So the hard point is kept as one bit
// per (variable, restart), 1/32 of the float row, and a step is two kernels:
//
//  * k_hard_prep draws the noise, decides x_hat and packs a wave's 64
//    decisions with a ballot;
//  * k_hard_update gathers the bit rows of a variable's occurrences, counts
//    them with bit-sliced adders (a lane adds 64 restarts at once), and
//    applies the soft backward and the optimizer in the same kernel, so the
//    gradient never goes to memory.
//
// Counts are exact integers below 2^8, so the results are those of summing
// the 0/1 products in FP64.
//
// What bounds it: the prep kernel the VALU (12 quarter-rate multiplies of the
// hash and the FP64 logarithm), the update kernel its seven float rows (4.0
// TB/s) and the FP64 update (65 % VALU busy) together; the gathers of the
// gradient are 1/32 of the float rows'.  Planted 3-SAT, Adam: n = 100,000 at
// 1,000 restarts 3260 us a step with the float passes, 1080 us with these
// (prep 475, update 700); n = 2,000 at 500 restarts 93 and 27 us.
//
// Taken by formulas (batches) whose variables all occur fewer than 256 times
// and whose longest clause is short for the restarts (hard_longest); the float
// passes run the others.
#include "galsat_device.h"

namespace galsat {

namespace {

// Occurrence records: x = own literal negated << 31 | first other code, y =
// first literal of its clause << 31 | second other code.  kNoCode: no such
// literal; y = kLongClause: a clause of more than 3 literals, x holds its id.
constexpr uint32_t kNoCode = 0x7fffffffu, kLongClause = 0x7ffffffeu;

__global__ __launch_bounds__(256) void k_hard_records(const int32_t* clause_ptr,
                                                      const int32_t* clause_lits, int32_t m,
                                                      const int32_t* var_ptr, int32_t* cursor,
                                                      uint2* rec) {
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < m; t += (int64_t)gridDim.x * 256) {
    const int cs = clause_ptr[t], ce = clause_ptr[t + 1], k = ce - cs;
    for (int p = cs; p < ce; ++p) {
      const uint32_t code = (uint32_t)clause_lits[p];
      uint2 o = make_uint2(kNoCode, kNoCode);
      if (k > 3) {
        o = make_uint2((uint32_t)t, kLongClause);
      } else {
        for (int i = cs; i < ce; ++i) {
          if (i == p) continue;
          if (o.x == kNoCode) o.x = (uint32_t)clause_lits[i];
          else o.y = (uint32_t)clause_lits[i];
        }
      }
      o.x |= (code & 1u) << 31;
      o.y |= p == cs ? 0x80000000u : 0u;
      const int v = (int)(code >> 1);
      rec[var_ptr[v] + atomicAdd(&cursor[v], 1)] = o;
    }
  }
}

// Hard point x_hat = [d + l > 0] (FP32 sum; a tie goes to state 0) of 64
// restarts a wave, packed; l is kept for the update.  noise: caller-given l
// (then not copied) or null to draw it.
__global__ __launch_bounds__(256) void k_hard_prep(const float* __restrict__ d, int32_t ldd,
                                                   const float* __restrict__ noise, uint64_t seed,
                                                   int32_t t, int32_t n, int32_t R, int32_t words,
                                                   uint64_t* __restrict__ bits,
                                                   float* __restrict__ nb, int32_t ldn) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int word = blockIdx.y, r = word * 64 + lane;
  const bool here = r < R;
  for (int64_t v = (int64_t)blockIdx.x * 4 + w; v < n; v += (int64_t)gridDim.x * 4) {
    float s = 0.0f;
    if (here) {
      const float dv = d[v * ldd + r];
      float l;
      if (noise) {
        l = noise[v * ldd + r];
      } else {
        l = gumbel_diff(seed, t, v, r);
        nb[v * ldn + r] = l;
      }
      s = dv + l;
    }
    const uint64_t m = __ballot(s > 0.0f);
    if (lane == 0) bits[v * words + word] = m;
  }
}

// planes += the four one-bit numbers m
template <int P>
__device__ __forceinline__ void add4(uint64_t (&c)[P], const uint64_t (&m)[4]) {
  uint64_t s, c1, c2, s0, s1, s2;
  full_add(m[0], m[1], m[2], s, c1);
  s0 = s ^ m[3];
  c2 = s & m[3];
  s1 = c1 ^ c2;
  s2 = c1 & c2;
  uint64_t carry = c[0] & s0;
  c[0] ^= s0;
  full_add(c[1], s1, carry, c[1], carry);
  full_add(c[2], s2, carry, c[2], carry);
#pragma unroll
  for (int p = 3; p < P; ++p) {
    const uint64_t t = c[p] & carry;
    c[p] ^= carry;
    carry = t;
  }
}

__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return (uint64_t)hi << 32 | lo;
}

// Counter of this lane's restart: the planes of lane src, whose 64 counters
// belong to the wave's 64 lanes.
template <int P>
__device__ __forceinline__ int lane_count(const uint64_t (&c)[P], int src) {
  int cnt = 0;
#pragma unroll
  for (int p = 0; p < P; ++p)
    cnt += __builtin_amdgcn_inverse_ballot_w64(lane_u64(c[p], src)) ? 1 << p : 0;
  return cnt;
}

__device__ __forceinline__ uint64_t false_mask(uint32_t code, uint64_t row) {
  return (code & 1u) ? row : ~row;
}

// Orders the LDS accesses of a wave's lanes before and after it.  The LDS
// serves a wave's instructions in order, so the fences only keep the compiler
// from moving an access across (the wave barrier alone does not: it is no
// memory access).
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave takes 16 / LW variables and LW words of 64 restarts: lane = variable
// * 4 LW + group * LW + word, group g counting occurrences g, g + 4, ...; its
// 16 (variable, word) pairs are then updated by all lanes, V restarts a lane
// and V pairs at a time.  P: planes of a variable's count (occurrences below
// 2^P).
template <int LW, int P, bool ADAM, int V>
__global__ __launch_bounds__(256) void k_hard_update(HardArgs a) {
  constexpr int NV = 16 / LW;
  constexpr int LP = 64 / V;  // lanes of a pair
  constexpr int UP = 6;       // planes of the unsat counters, emptied in time
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
  const int vs = lane / (4 * LW), g = lane / LW % 4, w = lane % LW;
  const int W = a.words, w0 = blockIdx.y * LW, wc = min(w0 + w, W - 1);
  const int vb = a.chunk[blockIdx.x].x, ve = a.chunk[blockIdx.x].y;
  __shared__ int s_cnt[LW * 64];
  __shared__ uint32_t s_plane[4][P][32];  // of each wave's pairs, low and high half
  __shared__ int s_npos[4][16];
  if (a.unsat_part) {
    for (int i = threadIdx.x; i < LW * 64; i += 256) s_cnt[i] = 0;
    __syncthreads();
  }
  uint64_t up[UP];
#pragma unroll
  for (int p = 0; p < UP; ++p) up[p] = 0;
  int room = (1 << UP) - 1;  // what the unsat counters can still take (uniform)
  // the lanes of a word are added first, so only LW lanes' planes are spread
  // over the restarts
  auto empty_unsat = [&]() {
    constexpr int TP = UP + ilog2(64 / LW);
    uint64_t all[TP];
#pragma unroll
    for (int p = 0; p < TP; ++p) all[p] = p < UP ? up[p] : 0;
#pragma unroll
    for (int off = LW; off < 64; off *= 2) add_lane<TP>(all, off);
#pragma unroll 1
    for (int src = 0; src < LW; ++src) {
      const int c = lane_count<TP>(all, src);
      if (c) atomicAdd(&s_cnt[src * 64 + lane], c);
    }
#pragma unroll
    for (int p = 0; p < UP; ++p) up[p] = 0;
    room = (1 << UP) - 1;
  };

  for (int base = vb + wv * NV; base < ve; base += 4 * NV) {
    const int v = base + vs < ve ? base + vs : ve - 1;
    const int q0 = a.var_ptr[v];
    const int dg = base + vs < ve ? a.var_ptr[v + 1] - q0 : 0;
    const uint64_t own = a.bits[(int64_t)v * W + wc];
    uint64_t c[P];
    int npos = 0;
#pragma unroll
    for (int p = 0; p < P; ++p) c[p] = 0;
    for (int i0 = g; __any(i0 < dg); i0 += 16) {
      uint2 rec[4];
      uint64_t b1[4], b2[4], m[4], un[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        rec[u] = make_uint2(kNoCode, kNoCode);
        if (i0 + 4 * u < dg) rec[u] = a.rec[q0 + i0 + 4 * u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t c1 = rec[u].x & kNoCode, c2 = rec[u].y & kNoCode;
        b1[u] = b2[u] = 0;
        if (c2 != kLongClause) {
          if (c1 != kNoCode) b1[u] = a.bits[(int64_t)(c1 >> 1) * W + wc];
          if (c2 != kNoCode) b2[u] = a.bits[(int64_t)(c2 >> 1) * W + wc];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t c1 = rec[u].x & kNoCode, c2 = rec[u].y & kNoCode;
        const bool here = i0 + 4 * u < dg, neg = (rec[u].x >> 31) != 0;
        uint64_t mask = ~0ULL;
        if (c2 == kLongClause) {
          // the clause's literals but one of the own code (if it is there
          // twice, the other one stays)
          const uint32_t oc = ((uint32_t)v << 1) | (neg ? 1u : 0u);
          bool skipped = false;
          for (int p = a.clause_ptr[c1]; p < a.clause_ptr[c1 + 1]; ++p) {
            const uint32_t code = (uint32_t)a.clause_lits[p];
            if (code == oc && !skipped) {
              skipped = true;
              continue;
            }
            mask &= false_mask(code, a.bits[(int64_t)(code >> 1) * W + wc]);
          }
        } else {
          if (c1 != kNoCode) mask &= false_mask(c1, b1[u]);
          if (c2 != kNoCode) mask &= false_mask(c2, b2[u]);
        }
        // a positive occurrence adds 1 - m here and -1 through npos
        m[u] = here ? (neg ? mask : ~mask) : 0;
        npos += here && !neg ? 1 : 0;
        un[u] = here && (rec[u].y >> 31) ? mask & (neg ? own : ~own) : 0;
      }
      add4<P>(c, m);
      if (a.unsat_part) {
        if (room < 4) empty_unsat();
        add4<UP>(up, un);
        room -= 4;
      }
    }
    add_lane<P>(c, LW);
    add_lane<P>(c, 2 * LW);
    npos += __shfl_xor(npos, LW, 64);
    npos += __shfl_xor(npos, 2 * LW, 64);

    // group 0 holds the totals: pair = variable * LW + word
    if (g == 0) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        s_plane[wv][p][2 * (vs * LW + w)] = (uint32_t)c[p];
        s_plane[wv][p][2 * (vs * LW + w) + 1] = (uint32_t)(c[p] >> 32);
      }
      s_npos[wv][vs * LW + w] = npos;
    }
    wave_sync_lds();

    // the next pairs' rows are loaded while these are computed
    float dn[V], ln[V], mn[V], vn[V];
    auto at = [&](int j, int64_t& v2, int& r) {
      v2 = base + j / LW;
      r = (w0 + j % LW) * 64 + lane % LP * V;
      return j < 16 && v2 < ve && r < a.R;
    };
    auto fetch = [&](int j) {
      int64_t v2;
      int r;
      if (at(j, v2, r)) {
        load_row<V>(a.d + v2 * a.ldd + r, dn);
        load_row<V>(a.noise + v2 * a.ldn + r, ln);
        if constexpr (ADAM) {
          load_row<V>(a.mom + v2 * a.ldd + r, mn);
          load_row<V>(a.vel + v2 * a.ldd + r, vn);
        }
      }
    };
    fetch(lane / LP);
#pragma unroll 1
    for (int j0 = 0; j0 < 16 && base + j0 / LW < ve; j0 += V) {
      const int j = j0 + lane / LP;
      float dj[V], lj[V], mj[V], vj[V];
#pragma unroll
      for (int e = 0; e < V; ++e) {
        dj[e] = dn[e];
        lj[e] = ln[e];
        mj[e] = mn[e];
        vj[e] = vn[e];
      }
      fetch(j + V);
      int64_t v2;
      int r;
      if (at(j, v2, r)) {
        // this lane's V bits of each plane, spread to the bytes of a word
        // that adds up the planes: one byte per restart
        const int half = 2 * j + (lane % LP) * V / 32;
        uint32_t bytes = 0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const uint32_t nib = (s_plane[wv][p][half] >> ((lane % LP) * V % 32)) & ((1u << V) - 1u);
          bytes += (V == 1 ? nib : __umul24(nib, 0x204081u) & 0x01010101u) << p;
        }
        const int less = s_npos[wv][j];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const int cnt = (int)(bytes >> (8 * e) & 255u) - less;
          dj[e] = gumbel_apply<ADAM>(dj[e], lj[e], (double)cnt, a.o, mj[e], vj[e]);
        }
        store_row<V>(a.d + v2 * a.ldd + r, dj);
        if constexpr (ADAM) {
          store_row<V>(a.mom + v2 * a.ldd + r, mj);
          store_row<V>(a.vel + v2 * a.ldd + r, vj);
        }
      }
    }
    wave_sync_lds();  // before the next variables' planes
  }
  if (a.unsat_part) {
    empty_unsat();
    __syncthreads();
    for (int i = threadIdx.x; i < LW * 64; i += 256) {
      const int r = w0 * 64 + i;
      if (r < a.R) a.unsat_part[(int64_t)blockIdx.x * a.R + r] = s_cnt[i];
    }
  }
}

template <int LW, int P, bool ADAM>
hipError_t hard_update_adam(const HardArgs& a, int chunks, hipStream_t s) {
  const dim3 grid(chunks, (a.words + LW - 1) / LW);
  // four restarts a lane where every row starts on 16 bytes and ends at four
  // restarts
  auto ok = [](const float* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  const bool wide = a.R % 4 == 0 && a.ldd % 4 == 0 && a.ldn % 4 == 0 && ok(a.d) && ok(a.noise) &&
                    (!ADAM || (ok(a.mom) && ok(a.vel)));
  if (wide) hipLaunchKernelGGL((k_hard_update<LW, P, ADAM, 4>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_hard_update<LW, P, ADAM, 1>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int LW, int P>
hipError_t hard_update_go(const HardArgs& a, int chunks, bool adam, hipStream_t s) {
  return adam ? hard_update_adam<LW, P, true>(a, chunks, s) : hard_update_adam<LW, P, false>(a, chunks, s);
}

template <int P>
hipError_t hard_update_p(const HardArgs& a, int lw, int chunks, bool adam, hipStream_t s) {
  switch (lw) {
    case 1: return hard_update_go<1, P>(a, chunks, adam, s);
    case 2: return hard_update_go<2, P>(a, chunks, adam, s);
    case 4: return hard_update_go<4, P>(a, chunks, adam, s);
    case 8: return hard_update_go<8, P>(a, chunks, adam, s);
    case 16: return hard_update_go<16, P>(a, chunks, adam, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int hard_lanes(int32_t R) {
  int lw = 1;
  while (lw < 16 && lw * 64 < R) lw *= 2;
  return lw;
}

hipError_t launch_hard_records(const int32_t* clause_ptr, const int32_t* clause_lits, int32_t m,
                               const int32_t* var_ptr, int32_t n, int32_t* cursor, uint2* rec,
                               hipStream_t s) {
  const hipError_t e = launch_zero_i32(cursor, n, s);
  if (e != hipSuccess || m <= 0) return e;
  hipLaunchKernelGGL(k_hard_records, dim3(grid_x_for(((int64_t)m + 255) / 256)), dim3(256), 0, s,
                     clause_ptr, clause_lits, m, var_ptr, cursor, rec);
  return hipGetLastError();
}

hipError_t launch_hard_prep(const float* d, int32_t ldd, const float* noise, uint64_t seed, int32_t t,
                            int32_t n, int32_t R, uint64_t* bits, float* nb, int32_t ldn,
                            hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int words = (R + 63) / 64;
  const int64_t rows = ((int64_t)n + 3) / 4;
  // about eight workgroups a CU, each wave walking many rows of one word
  const int64_t gx = std::min<int64_t>(rows, std::max<int64_t>(1, 8 * 256 * 4 / words));
  hipLaunchKernelGGL(k_hard_prep, dim3((uint32_t)gx, words), dim3(256), 0, s, d, ldd, noise, seed, t,
                     n, R, words, bits, nb, ldn);
  return hipGetLastError();
}

hipError_t launch_hard_update(const HardArgs& a, int chunks, int planes, bool adam, hipStream_t s) {
  if (chunks <= 0) return hipSuccess;
  const int lw = hard_lanes(a.R);
  return planes <= kHardPlanes ? hard_update_p<kHardPlanes>(a, lw, chunks, adam, s)
                               : hard_update_p<kHardPlanesMax>(a, lw, chunks, adam, s);
}

}  // namespace galsat
