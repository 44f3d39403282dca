// Persistent LDS schedule (gfx950): for formulas small enough that a
// restart group's state fits in LDS, one workgroup per (formula, restart
// group) runs every step of galsat_step in one launch.  The state is
// double-buffered in LDS (every variable updates from the same x_k:
// Jacobi); the formula's occurrence records and var_ptr slice are copied
// to LDS once per launch when they fit (else read from global memory), so
// a step touches global memory only for its trace entries.  Each step's
// loss' and rounded unsat count are reduced in a fixed order (wave
// butterflies, then the waves in index order).  The gradient of a variable
// is summed over its occurrences in var_occ order in FP64 from the same
// FP32 products as the variable pass (Section 3.2, Eq. 2 and its
// derivative), so states equal the general schedule's bitwise when no
// variable is split.
#include "galsat_device.h"

namespace galsat {

namespace {

constexpr int kPersistWaves = kPersistBlock / 64;

struct PersistLayout {
  size_t occ, red_l, red_u, vp, x, total;
};

// byte offsets of the dynamic LDS areas; records first (16-byte aligned)
__host__ __device__ inline PersistLayout persist_layout(int rg, int nf_max, int nocc_stage) {
  PersistLayout p;
  p.occ = 0;
  p.red_l = p.occ + (size_t)nocc_stage * 16;                           // double [2][waves][rg]
  p.red_u = p.red_l + (size_t)2 * kPersistWaves * rg * sizeof(double); // int [2][waves][rg]
  p.vp = p.red_u + (size_t)2 * kPersistWaves * rg * sizeof(int);      // int [nf_max + 1]
  p.x = p.vp + (((size_t)nf_max + 1) * sizeof(int) + 15) / 16 * 16;    // float [2][nf_max][rg]
  p.total = p.x + (size_t)2 * nf_max * rg * sizeof(float);
  return p;
}

template <int RG>
__device__ __forceinline__ float lds_row(const float* xs, int vb, int code, int lane) {
  return xs[((code >> 1) - vb) * RG + lane];
}

// STAGED picks where the records are read (LDS or global memory) at compile
// time, so that every load has one address space (no generic loads).
template <int RG, bool STAGED>
__global__ __launch_bounds__(kPersistBlock) void k_persistent(PersistArgs a) {
  constexpr int IPB = kPersistBlock / RG;
  extern __shared__ int4 smem4[];
  char* smem = reinterpret_cast<char*>(smem4);
  const PersistLayout lay = persist_layout(RG, a.nf_max, STAGED ? a.nocc_max : 0);
  int4* s_occ = reinterpret_cast<int4*>(smem + lay.occ);
  double* s_l = reinterpret_cast<double*>(smem + lay.red_l);
  int* s_u = reinterpret_cast<int*>(smem + lay.red_u);
  int* s_vp = reinterpret_cast<int*>(smem + lay.vp);
  float* xa = reinterpret_cast<float*>(smem + lay.x);
  float* xb = xa + (int64_t)a.nf_max * RG;
  const int groups = (a.R + RG - 1) / RG;
  const int f = a.f_order[blockIdx.x / groups], grp = blockIdx.x % groups;
  const int lane = threadIdx.x % RG, slot = threadIdx.x / RG;
  const int wave = threadIdx.x / 64, wlane = threadIdx.x % 64;
  const int r = grp * RG + lane;
  const bool active = r < a.R;
  const int vb = a.f_vbeg[f], nf = a.f_vbeg[f + 1] - vb;
  const int qb = a.var_ptr[vb];
  for (int i = threadIdx.x; i <= nf; i += kPersistBlock) s_vp[i] = a.var_ptr[vb + i] - qb;
  if constexpr (STAGED) {
    const int nocc = a.var_ptr[vb + nf] - qb;
    for (int i = threadIdx.x; i < nocc; i += kPersistBlock) s_occ[i] = a.occ[qb + i];
  }
  for (int i = threadIdx.x; i < nf * RG; i += kPersistBlock) {
    const int rr = grp * RG + i % RG;
    xa[i] = rr < a.R ? a.x[(int64_t)(vb + i / RG) * a.ldx + rr] : 0.0f;
  }
  __syncthreads();
  for (int k = 0; k < a.steps; ++k) {
    double lsum = 0.0;
    int usum = 0;
    for (int vi = slot; vi < nf; vi += IPB) {
      const float xv = xa[vi * RG + lane];
      double g = 0.0;
      const int q0 = s_vp[vi], q1 = s_vp[vi + 1];
      // one occurrence's contribution, in var_occ order (q is formula-local)
      auto add = [&](const int4 o, int q) {
        const int hdr = o.x, nother = rec_nother(hdr);
        const bool first = rec_first(hdr), neg = rec_neg(hdr);
        float prod = 1.0f;
        bool any_true = false;
        if (rec_kind(hdr) == kRecInline) {
          int codes[7] = {o.y, o.z, o.w, 0, 0, 0, 0};
          if (nother > 3) {
            const int4 e = a.occx[qb + q];
            codes[3] = e.x; codes[4] = e.y; codes[5] = e.z; codes[6] = e.w;
          }
#pragma unroll
          for (int c = 0; c < 7; ++c) {
            if (c < nother) {
              const float y = lds_row<RG>(xa, vb, codes[c], lane);
              prod *= lit_factor(codes[c], y);
              any_true = any_true || lit_true(codes[c], y);
            }
          }
        } else {  // GENERAL: the clause's other literals in clause order
          const int t = o.y, p = o.z;
          for (int i = a.clause_ptr[t]; i < a.clause_ptr[t + 1]; ++i) {
            if (i == p) continue;
            const int code = a.clause_lits[i];
            const float y = lds_row<RG>(xa, vb, code, lane);
            prod *= lit_factor(code, y);
            any_true = any_true || lit_true(code, y);
          }
        }
        g += (double)(neg ? prod : -prod);
        if (first) {
          const int own = neg ? 1 : 0;
          lsum += (double)(lit_factor(own, xv) * prod);
          usum += (any_true || lit_true(own, xv)) ? 0 : 1;
        }
      };
      // the same contribution for an inline record with at most three other
      // literals whose states are already read (an absent literal's factor
      // is exactly 1, so the product is the same)
      auto add3 = [&](const int4 o, const float* y) {
        const int hdr = o.x, nother = rec_nother(hdr);
        const bool first = rec_first(hdr), neg = rec_neg(hdr);
        const int codes[3] = {o.y, o.z, o.w};
        float prod = 1.0f;
        bool any_true = false;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const bool here = c < nother;
          prod *= here ? lit_factor(codes[c], y[c]) : 1.0f;
          any_true = any_true || (here && lit_true(codes[c], y[c]));
        }
        g += (double)(neg ? prod : -prod);
        if (first) {
          const int own = neg ? 1 : 0;
          lsum += (double)(lit_factor(own, xv) * prod);
          usum += (any_true || lit_true(own, xv)) ? 0 : 1;
        }
      };
      const int4* recs;
      if constexpr (STAGED) recs = s_occ;
      else recs = a.occ + qb;
      const int self = (vb + vi) << 1;  // a code whose state row is in LDS
      // four records in flight; a partial last batch re-reads its last
      // record and masks the extra contributions off
      for (int q = q0; q < q1; q += 4) {
        int4 o[4];
        bool ok[4];
#pragma unroll
        for (int k2 = 0; k2 < 4; ++k2) {
          ok[k2] = q + k2 < q1;
          o[k2] = recs[ok[k2] ? q + k2 : q1 - 1];
        }
        bool short3 = true;
#pragma unroll
        for (int k2 = 0; k2 < 4; ++k2)
          short3 = short3 && rec_kind(o[k2].x) == kRecInline && rec_nother(o[k2].x) <= 3;
        if (short3) {  // every state read of the four issued before any use
          float y[4][3];
#pragma unroll
          for (int k2 = 0; k2 < 4; ++k2) {
            const int nother = rec_nother(o[k2].x);
            y[k2][0] = lds_row<RG>(xa, vb, nother > 0 ? o[k2].y : self, lane);
            y[k2][1] = lds_row<RG>(xa, vb, nother > 1 ? o[k2].z : self, lane);
            y[k2][2] = lds_row<RG>(xa, vb, nother > 2 ? o[k2].w : self, lane);
          }
#pragma unroll
          for (int k2 = 0; k2 < 4; ++k2)
            if (ok[k2]) add3(o[k2], y[k2]);
        } else {
#pragma unroll
          for (int k2 = 0; k2 < 4; ++k2)
            if (ok[k2]) add(o[k2], q + k2);
        }
      }
      xb[vi * RG + lane] = clamp01((double)xv - (double)a.lr * g);
    }
    // fixed-order reduction over the slots of each restart: butterflies over
    // the wave's slots, then the waves in index order; buffers alternate by
    // step so one barrier per step suffices
#pragma unroll
    for (int off = RG; off < 64; off <<= 1) {
      lsum += __shfl_xor(lsum, off);
      usum += __shfl_xor(usum, off);
    }
    const int buf = (k & 1) * kPersistWaves * RG;
    if (wlane < RG) {
      s_l[buf + wave * RG + lane] = lsum;
      s_u[buf + wave * RG + lane] = usum;
    }
    float* tmp = xa;
    xa = xb;
    xb = tmp;
    __syncthreads();
    if (threadIdx.x < RG && active) {
      double tot = 0.0;
      int utot = 0;
#pragma unroll
      for (int w = 0; w < kPersistWaves; ++w) {
        tot += s_l[buf + w * RG + lane];
        utot += s_u[buf + w * RG + lane];
      }
      const int64_t o = ((int64_t)k * a.F + f) * a.R + r;
      if (a.loss_trace) a.loss_trace[o] = (float)(tot + (double)a.n_empty[f]);
      if (a.unsat_trace) a.unsat_trace[o] = utot + a.n_empty[f];
    }
  }
  for (int i = threadIdx.x; i < nf * RG; i += kPersistBlock) {
    const int rr = grp * RG + i % RG;
    if (rr < a.R) a.x[(int64_t)(vb + i / RG) * a.ldx + rr] = xa[i];
  }
}

}  // namespace

size_t persist_lds_bytes(int rg, int nf_max, int nocc_stage) {
  return persist_layout(rg, nf_max, nocc_stage).total;
}

hipError_t launch_persistent(const PersistArgs& a, int rg, hipStream_t s) {
  if (a.F <= 0 || a.steps <= 0) return hipSuccess;
  const int groups = (a.R + rg - 1) / rg;
  const size_t bytes = persist_lds_bytes(rg, a.nf_max, a.stage_occ ? a.nocc_max : 0);
  dim3 grid(a.F * groups), block(kPersistBlock);
#define GALSAT_PERSIST_CASE(N)                                                          \
  case N:                                                                               \
    if (a.stage_occ) hipLaunchKernelGGL((k_persistent<N, true>), grid, block, bytes, s, a); \
    else hipLaunchKernelGGL((k_persistent<N, false>), grid, block, bytes, s, a);            \
    break;
  switch (rg) {
    GALSAT_PERSIST_CASE(1)
    GALSAT_PERSIST_CASE(2)
    GALSAT_PERSIST_CASE(4)
    GALSAT_PERSIST_CASE(8)
    GALSAT_PERSIST_CASE(16)
    GALSAT_PERSIST_CASE(32)
    default: return hipErrorInvalidValue;
  }
#undef GALSAT_PERSIST_CASE
  return hipGetLastError();
}

// Clause-parallel form.  The kernel above gives each variable one thread,
// which walks the variable's occurrences one after another: at n = 200 and
// one restart per workgroup 312 of 512 threads have no variable, and the
// time of a step (6.9 us) is the longest variable's chain of LDS reads.
// Here a step is two short parallel phases with a barrier after each:
//
//  * a thread per clause reads the clause's literals once, forms every
//    literal's partial product and writes it to the literal's own slot, and
//    holds U_t and the rounded count;
//  * a thread per variable adds its slots in FP64.
//
// Clauses of up to three literals stay in registers for the whole launch
// (three words each: position code and slot of a literal); a missing literal
// names position nf, whose state is 0, so its factor is exactly 1, and the
// slot nobody reads.  Clauses of 4 to 8 literals are read from memory each
// step.  Variables are taken by decreasing occurrence count and their slots
// laid out by slices of 64 (slot j of lane l at base + 64 j + l), so the
// second phase reads LDS without conflicts and the lanes of a wave loop
// alike; slots past a variable's count hold 0.
//
// A product is formed in clause order skipping the own literal and a
// variable's sum runs in var_occ order in FP64, as in the kernel above, so
// the states are bitwise the same.  The loss is added per thread, then over
// the threads in a fixed order by the last wave while the other waves add
// variables.
//
// What bounds a step: the LDS latency of the two phases and two barriers.
// Planted 3-SAT of 200 variables at 64 restarts, 50 steps in a call: 319 us
// with the kernel above, 60 us with this one; a 10-step call of the general
// schedule (replayed from a graph) took 132 us and takes 17 us here.
namespace {

struct ClauseLdsLayout {
  size_t l, u, x, d, total;
};

__host__ __device__ inline ClauseLdsLayout clause_lds_layout(int threads, int32_t nf_max,
                                                             int32_t slot_max) {
  ClauseLdsLayout p;
  p.l = 0;                                                    // double [threads]
  p.u = p.l + (size_t)threads * sizeof(double);               // int [waves]
  p.x = p.u + (size_t)(threads / 64) * sizeof(int);           // float [nf_max + 1]
  p.d = p.x + (((size_t)nf_max + 1) * sizeof(float) + 15) / 16 * 16;  // float [slot_max + 1]
  p.total = p.d + ((size_t)slot_max + 1) * sizeof(float);
  return p;
}

__device__ __forceinline__ float pos_factor(uint32_t w, float y) {
  return (w & 1u) ? y : 1.0f - y;
}

__device__ __forceinline__ bool pos_true(uint32_t w, float y) {
  return (y > 0.5f) != ((w & 1u) != 0);
}

// Lane 63's value is the sum over the wave, added in a fixed order by DPP
// moves (a butterfly of shuffles goes through LDS six times, which took
// longer than the phase it runs beside).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return v + __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_total(double v) {
  v = dpp_add<0xb1, 0xf>(v);   // lane ^ 1
  v = dpp_add<0x4e, 0xf>(v);   // lane ^ 2
  v = dpp_add<0x141, 0xf>(v);  // half rows mirrored
  v = dpp_add<0x140, 0xf>(v);  // rows mirrored: each lane its row's sum
  v = dpp_add<0x142, 0xa>(v);  // row 0 into 1, row 2 into 3
  return dpp_add<0x143, 0xc>(v);  // rows 0 and 1 into 3
}

template <int T, int PER>
__global__ __launch_bounds__(T) void k_clause_lds(ClauseLdsArgs a) {
  constexpr int W = T / 64;
  constexpr int KL = kClauseLdsMaxLen;
  extern __shared__ int4 smem4[];
  char* smem = reinterpret_cast<char*>(smem4);
  const ClauseLdsLayout lay = clause_lds_layout(T, a.nf_max, a.slot_max);
  double* s_l = reinterpret_cast<double*>(smem + lay.l);
  int* s_u = reinterpret_cast<int*>(smem + lay.u);
  float* xs = reinterpret_cast<float*>(smem + lay.x);
  float* sd = reinterpret_cast<float*>(smem + lay.d);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  int row = blockIdx.x / a.R, r = blockIdx.x % a.R;
  if (a.xcd) {
    // consecutive workgroups go to the 8 XCDs in turn: a formula's restarts
    // stay on one XCD, whose L2 then holds the formula's state rows
    row = (blockIdx.x / (8 * a.R)) * 8 + blockIdx.x % 8;
    r = (blockIdx.x / 8) % a.R;
  }
  if (row >= a.F) return;  // the whole workgroup
  const int f = a.f_order[row];
  const int vb = a.f_vbeg[f], nf = a.f_vbeg[f + 1] - vb;
  const int sl0 = a.f_slice[f], nsl = a.f_slice[f + 1] - sl0;
  const int cs = a.f_short[f], ms = a.f_short[f + 1] - cs;
  const int cl = a.f_long[f], ml = a.f_long[f + 1] - cl;
  const uint32_t none = ((uint32_t)nf << 1) | ((uint32_t)a.slot_max << 16);
  uint32_t rec[PER][3];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int t = tid + i * T;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      rec[i][c] = t < ms ? a.short_rec[(int64_t)c * a.n_short + cs + t] : none;
  }
  for (int i = tid; i < nf; i += T) xs[i] = a.x[(int64_t)a.var[vb + i] * a.ldx + r];
  if (tid == 0) xs[nf] = 0.0f;
  for (int i = tid; i < a.slot_max; i += T) sd[i] = 0.0f;
  int2 first = make_int2(0, 0);
  if (wave < nsl) first = a.slice[sl0 + wave];
  const bool traced = a.loss_trace || a.unsat_trace;
  const int n_empty = a.n_empty[f];
  __syncthreads();
  for (int k = 0; k < a.steps; ++k) {
    double lsum = 0.0;
    int cnt = 0;  // unsatisfied clauses of the wave (uniform)
    float y[PER][3];
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
      for (int c = 0; c < 3; ++c) y[i][c] = xs[(rec[i][c] & 0xffffu) >> 1];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const uint32_t w0 = rec[i][0], w1 = rec[i][1], w2 = rec[i][2];
      const float f0 = pos_factor(w0, y[i][0]), f1 = pos_factor(w1, y[i][1]),
                  f2 = pos_factor(w2, y[i][2]);
      const float p0 = f1 * f2, p1 = f0 * f2, p2 = f0 * f1;
      sd[w0 >> 16] = (w0 & 1u) ? p0 : -p0;
      sd[w1 >> 16] = (w1 & 1u) ? p1 : -p1;
      sd[w2 >> 16] = (w2 & 1u) ? p2 : -p2;
      if (traced) {
        const bool here = tid + i * T < ms;
        lsum += here ? (double)(f0 * p0) : 0.0;
        const bool sat = pos_true(w0, y[i][0]) || pos_true(w1, y[i][1]) || pos_true(w2, y[i][2]);
        cnt += __popcll(__ballot(here && !sat));
      }
    }
    for (int base = 0; base < ml; base += T) {
      const bool here = base + tid < ml;
      uint32_t w[KL];
      float fa[KL];
      bool sat = false;
#pragma unroll
      for (int c = 0; c < KL; ++c)
        w[c] = here ? a.long_rec[(int64_t)c * a.n_long + cl + base + tid] : none;
#pragma unroll
      for (int c = 0; c < KL; ++c) fa[c] = xs[(w[c] & 0xffffu) >> 1];
#pragma unroll
      for (int c = 0; c < KL; ++c) {
        sat = sat || pos_true(w[c], fa[c]);
        fa[c] = pos_factor(w[c], fa[c]);
      }
      float pre = 1.0f;  // product of the literals before c
#pragma unroll
      for (int c = 0; c < KL; ++c) {
        float p = pre;
#pragma unroll
        for (int e = c + 1; e < KL; ++e) p *= fa[e];
        sd[w[c] >> 16] = (w[c] & 1u) ? p : -p;
        if (c == 0) lsum += here ? (double)(fa[0] * p) : 0.0;
        pre *= fa[c];
      }
      cnt += __popcll(__ballot(here && !sat));
    }
    if (traced) {
      s_l[tid] = lsum;
      if (lane == 0) s_u[wave] = cnt;
    }
    __syncthreads();
    for (int s = wave; s < nsl; s += W) {
      const int2 sl = s == wave ? first : a.slice[sl0 + s];
      const int v = s * 64 + lane;
      const float* col = sd + sl.x + lane;
      double g = 0.0;
      // the next slots are read while these are added (the last trip reads
      // its own again); a slice of variables without occurrences has none
      float nxt[kSliceUnroll];
#pragma unroll
      for (int u = 0; u < kSliceUnroll; ++u) nxt[u] = sl.y > 0 ? col[u * 64] : 0.0f;
      for (int j = 0; j < sl.y; j += kSliceUnroll) {
        float d[kSliceUnroll];
        const int jn = j + kSliceUnroll < sl.y ? j + kSliceUnroll : j;
#pragma unroll
        for (int u = 0; u < kSliceUnroll; ++u) d[u] = nxt[u];
#pragma unroll
        for (int u = 0; u < kSliceUnroll; ++u) nxt[u] = col[(jn + u) * 64];
#pragma unroll
        for (int u = 0; u < kSliceUnroll; ++u) g += (double)d[u];
      }
      if (v < nf) xs[v] = clamp01((double)xs[v] - (double)a.lr * g);
    }
    if (traced && wave == W - 1) {
      double tot = 0.0;
#pragma unroll
      for (int w = 0; w < W; ++w) tot += s_l[w * 64 + lane];
      int utot = 0;
#pragma unroll
      for (int w = 0; w < W; ++w) utot += s_u[w];
      tot = wave_total(tot);
      if (lane == 63) {
        const int64_t o = ((int64_t)k * a.F + f) * a.R + r;
        if (a.loss_trace) a.loss_trace[o] = (float)(tot + (double)n_empty);
        if (a.unsat_trace) a.unsat_trace[o] = utot + n_empty;
      }
    }
    __syncthreads();
  }
  for (int i = tid; i < nf; i += T) a.x[(int64_t)a.var[vb + i] * a.ldx + r] = xs[i];
}

}  // namespace

// Threads: four waves while that holds the short clauses twice over or
// less, then more threads before more clauses per thread, and never fewer
// than a quarter of the variables.
bool clause_lds_shape(int32_t short_max, int32_t nf_max, int* threads, int* per) {
  int t = 256;
  while (t < kClauseLdsMaxThreads && (short_max > 2 * t || nf_max > 4 * t)) t *= 2;
  int p = 2;
  while (p < kClauseLdsMaxPer && short_max > p * t) p *= 2;
  if (short_max > p * t) return false;
  *threads = t;
  *per = p;
  return true;
}

size_t clause_lds_bytes(int threads, int32_t nf_max, int32_t slot_max) {
  return clause_lds_layout(threads, nf_max, slot_max).total;
}

namespace {

template <int T, int PER>
hipError_t clause_lds_go(const ClauseLdsArgs& a, hipStream_t s) {
  const size_t bytes = clause_lds_bytes(T, a.nf_max, a.slot_max);
  // beyond 64 KiB dynamic LDS has to be allowed for the kernel; always the
  // same amount, as handles of other sizes may launch it from other threads
  if (bytes > (size_t)(64 << 10)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_clause_lds<T, PER>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerBlock);
    if (e != hipSuccess) return e;
  }
  const int64_t blocks = (int64_t)(a.xcd ? (a.F + 7) / 8 * 8 : a.F) * a.R;
  hipLaunchKernelGGL((k_clause_lds<T, PER>), dim3((uint32_t)blocks), dim3(T), bytes, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_clause_lds(const ClauseLdsArgs& a, int threads, int per, hipStream_t s) {
  if (a.F <= 0 || a.steps <= 0) return hipSuccess;
  switch (threads * 16 + per) {
    case 256 * 16 + 2: return clause_lds_go<256, 2>(a, s);
    case 512 * 16 + 2: return clause_lds_go<512, 2>(a, s);
    case 1024 * 16 + 2: return clause_lds_go<1024, 2>(a, s);
    case 1024 * 16 + 4: return clause_lds_go<1024, 4>(a, s);
    case 1024 * 16 + 8: return clause_lds_go<1024, 8>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace galsat
