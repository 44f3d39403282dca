// Clause pass, fixed-order reductions, state init / copy and the exact
// rounded unsat count of the general schedule (gfx950).
//
// Paper passages: clause value U_t = prod_i (1 - s_i) (Section 3.2, Eq. 2)
// with the negation rule of Eq. (1); loss' = sum_t U_t (Eq. 5 shifted by
// the clause count); rounding x_hat = [x > 0.5] is the argmax of Eq. (4)
// with ties to 0.
#include "galsat_device.h"

namespace galsat {

// -------------------------------------------------------- clause pass
//
// For each clause t of the chunk: U_t = prod_i factor_i, its rounded
// satisfaction, and the partial of every literal j,
//   D[slot(j)][r] = slope_j * prod_{i<j} factor_i * prod_{i>j} factor_i,
// from a forward prefix sweep (prefix stored in place) and a backward
// suffix sweep.  No division: exact zero factors need no special case.
template <int LPI, int RPL>
__global__ __launch_bounds__(kBlock) void k_clause_pass(ClausePassArgs a) {
  constexpr int IPB = kBlock / LPI;
  constexpr int RT = LPI * RPL;
  const int lane = threadIdx.x % LPI, slot = threadIdx.x / LPI;
  const int chunk =
      a.chunk_order ? ldc(a.chunk_order, a.chunk_base + blockIdx.x) : a.chunk_base + blockIdx.x;
  if (chunk < 0) return;  // padding of the XCD-aware order: the whole block leaves
  const int tile = a.tile_base + blockIdx.y;
  const int r0 = tile * RT + lane * RPL;
  const bool active = r0 < a.R;
  const int rc = active ? r0 : 0;  // in-bounds column for lanes past the last restart
  const int cb = ldc(a.chunk_cbeg, chunk), ce = ldc(a.chunk_cend, chunk);
  double lsum[RPL];
  int usum[RPL];
#pragma unroll
  for (int j = 0; j < RPL; ++j) { lsum[j] = 0.0; usum[j] = 0; }

  for (int c0 = cb + slot; c0 < ce; c0 += IPB) {
    const int t = uniform<LPI>(a.clause_ids ? ldc(a.clause_ids, c0) : c0);
    const int s = ldc(a.clause_ptr, t), e = ldc(a.clause_ptr, t + 1);
    float pre[RPL];
    bool any_true[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) { pre[j] = 1.0f; any_true[j] = false; }
    // forward sweep, four literals' rows in flight at a time; with WRITE_D
    // the prefix product before each literal is stored in its partial row
    int i = s;
    for (; i + 4 <= e; i += 4) {
      int code[4];
      float y[4][RPL];
#pragma unroll
      for (int u = 0; u < 4; ++u) code[u] = ldc(a.clause_lits, i + u);
#pragma unroll
      for (int u = 0; u < 4; ++u) load_row<RPL>(a.x + (int64_t)(code[u] >> 1) * a.ldx + rc, y[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (active) store_row<RPL>(a.D + (int64_t)ldc(a.lit_dslot, i + u) * a.ldD + r0, pre);
#pragma unroll
        for (int j = 0; j < RPL; ++j) {
          pre[j] *= lit_factor(code[u], y[u][j]);
          any_true[j] = any_true[j] || lit_true(code[u], y[u][j]);
        }
      }
    }
    for (; i < e; ++i) {
      const int code = ldc(a.clause_lits, i);
      float y[RPL];
      load_row<RPL>(a.x + (int64_t)(code >> 1) * a.ldx + rc, y);
      if (active) store_row<RPL>(a.D + (int64_t)ldc(a.lit_dslot, i) * a.ldD + r0, pre);
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        pre[j] *= lit_factor(code, y[j]);
        any_true[j] = any_true[j] || lit_true(code, y[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < RPL; ++j) {
      lsum[j] += (double)pre[j];
      usum[j] += any_true[j] ? 0 : 1;
    }
    // backward sweep: partial = slope * prefix * suffix
    float suf[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) suf[j] = 1.0f;
    int i2 = e - 1;
    for (; i2 - 3 >= s; i2 -= 4) {
      int code[4];
      float y[4][RPL], d[4][RPL];
#pragma unroll
      for (int u = 0; u < 4; ++u) code[u] = ldc(a.clause_lits, i2 - u);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        load_row<RPL>(a.x + (int64_t)(code[u] >> 1) * a.ldx + rc, y[u]);
        load_row<RPL>(a.D + (int64_t)ldc(a.lit_dslot, i2 - u) * a.ldD + rc, d[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float slope = (code[u] & 1) ? 1.0f : -1.0f;
#pragma unroll
        for (int j = 0; j < RPL; ++j) {
          d[u][j] = slope * (d[u][j] * suf[j]);
          suf[j] *= lit_factor(code[u], y[u][j]);
        }
        if (active) store_row<RPL>(a.D + (int64_t)ldc(a.lit_dslot, i2 - u) * a.ldD + r0, d[u]);
      }
    }
    for (; i2 >= s; --i2) {
      const int code = ldc(a.clause_lits, i2);
      float y[RPL], d[RPL];
      load_row<RPL>(a.x + (int64_t)(code >> 1) * a.ldx + rc, y);
      float* dp = a.D + (int64_t)ldc(a.lit_dslot, i2) * a.ldD;
      load_row<RPL>(dp + rc, d);
      const float slope = (code & 1) ? 1.0f : -1.0f;
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        d[j] = slope * (d[j] * suf[j]);
        suf[j] *= lit_factor(code, y[j]);
      }
      if (active) store_row<RPL>(dp + r0, d);
    }
  }
  block_partials<LPI, RPL>(lsum, usum, a.chunk_row ? ldc(a.chunk_row, chunk) : chunk, tile, a.R,
                           a.loss_part, a.unsat_part);
}

// ---------------------------------------------------------- loss only
//
// Sum of U_t = prod_i factor_i over the chunk's clauses, nothing stored and
// no counts.  An item slot takes C consecutive clauses a trip: their first
// three literals' codes, then those rows, all in flight (the clause pass above
// walks a 3-literal clause one literal at a time), then what longer clauses
// have left: four at a time, and EXACT: the last one to three one by one (else
// the last four positions repeat the clause's last literal).  A product runs
// in clause order.  launch_loss_pass has the rule for C and EXACT.
// The list is sorted by each clause's most frequent variable where the state
// does not fit the caches, so that variable's row is gathered once for
// several clauses; a.xcd_pin maps restart tiles to XCDs as in k_var_pass.
// What bounds it: the gathers from beyond the L2 (6.5 TB/s).  Planted 3-SAT,
// the whole call with the clause pass and with this kernel: n = 100,000 x 1,024
// restarts 1,206 and 539 us, 50,001 x 250 137 and 92 us, 10,000 x 500 68 and 40 us.
template <int LPI, int RPL, int C, bool EXACT>
__global__ __launch_bounds__(kBlock) void k_loss_pass(ClausePassArgs a) {
  constexpr int IPB = kBlock / LPI;
  constexpr int RT = LPI * RPL;
  constexpr int H = 3;
  const int lane = threadIdx.x % LPI, slot = threadIdx.x / LPI;
  int chunk = blockIdx.x, tile = blockIdx.y;
  if (a.xcd_pin) {
    const int lin = blockIdx.y * gridDim.x + blockIdx.x;
    tile = lin % gridDim.y;
    chunk = lin / gridDim.y;
  }
  const int chunks = gridDim.x;
  const int r0 = tile * RT + lane * RPL;
  const int rc = r0 < a.R ? r0 : 0;  // in-bounds column for lanes past the last restart
  const int cb = a.chunk_cbeg ? ldc(a.chunk_cbeg, chunk) : (int)((int64_t)a.list_len * chunk / chunks);
  const int ce = a.chunk_cbeg ? ldc(a.chunk_cend, chunk) : (int)((int64_t)a.list_len * (chunk + 1) / chunks);
  const float* x = a.x + rc;
  double lsum[RPL];
  int usum[RPL];
#pragma unroll
  for (int j = 0; j < RPL; ++j) { lsum[j] = 0.0; usum[j] = 0; }
  // the factor as one FMA, exactly y or 1 - y
  auto factor = [](int code, float y) {
    return fmaf(y, (code & 1) ? 1.0f : -1.0f, (code & 1) ? 0.0f : 1.0f);
  };
  for (int c0 = cb + slot * C; c0 < ce; c0 += IPB * C) {
    const int c = uniform<LPI>(c0);
    int p[C + 1], code[C][H];
    float y[C][H][RPL];
#pragma unroll
    for (int k = 0; k <= C; ++k) p[k] = ldc(a.clause_ptr, min(c + k, ce));
#pragma unroll
    for (int k = 0; k < C; ++k)
      if (p[k + 1] > p[k]) {
#pragma unroll
        for (int h = 0; h < H; ++h) code[k][h] = ldc(a.clause_lits, min(p[k] + h, p[k + 1] - 1));
      }
#pragma unroll
    for (int k = 0; k < C; ++k)
      if (p[k + 1] > p[k]) {
#pragma unroll
        for (int h = 0; h < H; ++h) load_row<RPL>(x + (int64_t)(code[k][h] >> 1) * a.ldx, y[k][h]);
      }
#pragma unroll
    for (int k = 0; k < C; ++k) {
      float pre[RPL];
#pragma unroll
      for (int j = 0; j < RPL; ++j) pre[j] = 1.0f;
      if (p[k + 1] > p[k]) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const bool use = p[k] + h < p[k + 1];
#pragma unroll
          for (int j = 0; j < RPL; ++j) pre[j] *= use ? factor(code[k][h], y[k][h][j]) : 1.0f;
        }
        int i = p[k] + H;
        for (; EXACT ? i + 4 <= p[k + 1] : i < p[k + 1]; i += 4) {
          int cd[4];
          float z[4][RPL];
#pragma unroll
          for (int u = 0; u < 4; ++u) cd[u] = ldc(a.clause_lits, min(i + u, p[k + 1] - 1));
#pragma unroll
          for (int u = 0; u < 4; ++u) load_row<RPL>(x + (int64_t)(cd[u] >> 1) * a.ldx, z[u]);
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < RPL; ++j) pre[j] *= i + u < p[k + 1] ? factor(cd[u], z[u][j]) : 1.0f;
        }
        if constexpr (EXACT) {
          for (; i < p[k + 1]; ++i) {
            const int cd = ldc(a.clause_lits, i);
            float z[RPL];
            load_row<RPL>(x + (int64_t)(cd >> 1) * a.ldx, z);
#pragma unroll
            for (int j = 0; j < RPL; ++j) pre[j] *= factor(cd, z[j]);
          }
        }
      }
      if (c + k < ce) {
#pragma unroll
        for (int j = 0; j < RPL; ++j) lsum[j] += (double)pre[j];
      }
    }
  }
  block_partials<LPI, RPL>(lsum, usum, chunk, tile, a.R, a.loss_part, a.unsat_part);
}

// The list sorted by each clause's most frequent variable: a counting sort
// whose buckets (one per variable; clauses without literals last) are filled
// by atomics and then put in order by clause id, so the list does not depend
// on the order of the atomics.
namespace {

__global__ __launch_bounds__(256) void k_list_own(const int32_t* clause_ptr, const int32_t* clause_lits,
                                                  int32_t m, const int32_t* var_ptr, int32_t n,
                                                  int32_t* own, int32_t* count) {
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < m; t += (int64_t)gridDim.x * 256) {
    int best = n, most = 0;
    for (int i = clause_ptr[t]; i < clause_ptr[t + 1]; ++i) {
      const int v = clause_lits[i] >> 1, f = var_ptr[v + 1] - var_ptr[v];
      if (f > most) {
        best = v;
        most = f;
      }
    }
    own[t] = best;
    atomicAdd(&count[best], 1);
  }
}

// Exclusive prefix sums in place, one workgroup.
constexpr int kScanU = 16;
__global__ __launch_bounds__(1024) void k_list_scan(int32_t* a, int64_t len) {
  __shared__ int wave_tot[16], s_run;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) s_run = 0;
  __syncthreads();
  for (int64_t base = 0; base < len; base += 1024 * kScanU) {
    const int64_t i0 = base + (int64_t)tid * kScanU;
    int v[kScanU], sum = 0;
#pragma unroll
    for (int u = 0; u < kScanU; ++u) {
      v[u] = i0 + u < len ? a[i0 + u] : 0;
      sum += v[u];
    }
    int incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(incl, d, 64);
      if (lane >= d) incl += y;
    }
    if (lane == 63) wave_tot[w] = incl;
    __syncthreads();
    int before = s_run + incl - sum;
    for (int u = 0; u < w; ++u) before += wave_tot[u];
#pragma unroll
    for (int u = 0; u < kScanU; ++u) {
      if (i0 + u < len) a[i0 + u] = before;
      before += v[u];
    }
    __syncthreads();
    if (tid == 1023) s_run = before;
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_list_place(const int32_t* own, int32_t m, const int32_t* first,
                                                    int32_t* cursor, int32_t* ids) {
  for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < m; t += (int64_t)gridDim.x * 256)
    ids[first[own[t]] + atomicAdd(&cursor[own[t]], 1)] = (int32_t)t;
}

// A variable owns at most its occurrences, fewer than 256 here.
__global__ __launch_bounds__(256) void k_list_order(const int32_t* first, const int32_t* cursor, int32_t n,
                                                    int32_t* ids) {
  for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < n; v += (int64_t)gridDim.x * 256) {
    const int b = first[v], e = b + cursor[v];
    for (int i = b + 1; i < e; ++i) {
      const int x = ids[i];
      int j = i;
      for (; j > b && ids[j - 1] > x; --j) ids[j] = ids[j - 1];
      ids[j] = x;
    }
  }
}

__global__ __launch_bounds__(256) void k_list_lengths(const int32_t* clause_ptr, const int32_t* ids,
                                                      int32_t m, int32_t* len) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i <= m; i += (int64_t)gridDim.x * 256)
    len[i] = i < m ? clause_ptr[ids[i] + 1] - clause_ptr[ids[i]] : 0;
}

__global__ __launch_bounds__(256) void k_list_copy(const int32_t* clause_ptr, const int32_t* clause_lits,
                                                   const int32_t* ids, int32_t m, const int32_t* ptr,
                                                   int32_t* lits) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256) {
    const int s = clause_ptr[ids[i]], k = clause_ptr[ids[i] + 1] - s, o = ptr[i];
    for (int j = 0; j < k; ++j) lits[o + j] = clause_lits[s + j];
  }
}

}  // namespace

// ---------------------------------------------- short-clause partials
//
// Stored clauses of at most KS literals, one item (LPI lanes) per clause,
// read from the class's packed table (codes and D rows, -1 marking unused
// positions): the clause's rows are gathered once into registers, the
// exclusive prefix and suffix products formed there, and every literal's
// partial
//   slope_j * prefix_j * suffix_j
// written to its row of D.  One gather and one store per literal.
template <int LPI, int RPL, int KS>
__global__ __launch_bounds__(kBlock) void k_short_clause(ClausePassArgs a) {
  constexpr int IPB = kBlock / LPI;
  constexpr int RT = LPI * RPL;
  const int lane = threadIdx.x % LPI, slot = threadIdx.x / LPI;
  const int chunk =
      a.chunk_order ? ldc(a.chunk_order, a.chunk_base + blockIdx.x) : a.chunk_base + blockIdx.x;
  if (chunk < 0) return;  // padding of the XCD-aware order: the whole block leaves
  const int tile = a.tile_base + blockIdx.y;
  const int r0 = tile * RT + lane * RPL;
  const bool active = r0 < a.R;
  const int rc = active ? r0 : 0;
  const int cb = ldc(a.chunk_cbeg, chunk), ce = ldc(a.chunk_cend, chunk);
  double lsum[RPL];
  int usum[RPL];
#pragma unroll
  for (int j = 0; j < RPL; ++j) { lsum[j] = 0.0; usum[j] = 0; }

  for (int c0 = cb + slot; c0 < ce; c0 += IPB) {
    // the class's packed table: the clause's codes and D rows side by side,
    // so its row gathers depend on one table load only
    const int32_t* pk = a.packed + (int64_t)uniform<LPI>(c0) * 2 * KS;
    int code[KS], drow[KS];
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      code[u] = ldc(pk, u);
      drow[u] = ldc(pk, KS + u);
    }
    float f[KS][RPL];
    bool any_true[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) any_true[j] = false;
#pragma unroll
    for (int u = 0; u < KS; ++u) {
      const bool in = drow[u] >= 0;
      float y[RPL];
      if (in) {
        load_row<RPL>(a.x + (int64_t)(code[u] >> 1) * a.ldx + rc, y);
      } else {
#pragma unroll
        for (int j = 0; j < RPL; ++j) y[j] = 0.0f;  // factor 1 below
      }
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        f[u][j] = in ? lit_factor(code[u], y[j]) : 1.0f;
        any_true[j] = any_true[j] || (in && lit_true(code[u], y[j]));
      }
    }
    float pre[KS][RPL];
    float run[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) run[j] = 1.0f;
#pragma unroll
    for (int u = 0; u < KS; ++u)
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        pre[u][j] = run[j];
        run[j] *= f[u][j];
      }
#pragma unroll
    for (int j = 0; j < RPL; ++j) {
      lsum[j] += (double)run[j];
      usum[j] += any_true[j] ? 0 : 1;
    }
    float suf[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) suf[j] = 1.0f;
#pragma unroll
    for (int u = KS - 1; u >= 0; --u) {
      float dv[RPL];
      const float slope = (code[u] & 1) ? 1.0f : -1.0f;
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        dv[j] = slope * (pre[u][j] * suf[j]);
        suf[j] *= f[u][j];
      }
      if (active && drow[u] >= 0) store_row<RPL>(a.D + (int64_t)drow[u] * a.ldD + r0, dv);
    }
  }
  block_partials<LPI, RPL>(lsum, usum, a.chunk_row ? ldc(a.chunk_row, chunk) : chunk, tile, a.R,
                           a.loss_part, a.unsat_part);
}

// ------------------------------------------------ wave-per-clause pass
//
// Stored clauses of G..KMAX literals, one wavefront per clause: the wave's
// 64 lanes form G = 64 / LPI literal groups of LPI lanes, each group
// covering the tile's restarts, and group g takes the clause's literals
// [g * m, g * m + m) with m = ceil(k / G) <= MAXC.  Every literal's row is
// gathered once and its factor kept in registers; a lane forms the prefix
// and suffix products within its run serially, and one exclusive scan of
// the run products across the groups (shuffles by multiples of LPI lanes,
// so a lane only combines values of its own restarts) supplies the
// products of the runs before and after.  The partial of literal j is
//   slope_j * (before * prefix_in_run) * (suffix_in_run * after),
// written to its row of D: one gather and one store per literal, nothing
// stored in between.  No division: exact zero factors need no special case.
template <int LPI, int RPL, int MAXC>
__global__ __launch_bounds__(kBlock) void k_wave_clause(ClausePassArgs a) {
  constexpr int G = 64 / LPI;
  constexpr int RT = LPI * RPL;
  constexpr int WPB = kBlock / 64;
  const int wave = threadIdx.x / 64, lw = threadIdx.x % 64;
  const int grp = lw / LPI, lane = lw % LPI;
  const int chunk =
      a.chunk_order ? ldc(a.chunk_order, a.chunk_base + blockIdx.x) : a.chunk_base + blockIdx.x;
  if (chunk < 0) return;  // padding of the XCD-aware order: the whole block leaves
  const int tile = a.tile_base + blockIdx.y;
  const int r0 = tile * RT + lane * RPL;
  const bool active = r0 < a.R;
  const int rc = active ? r0 : 0;
  const int cb = ldc(a.chunk_cbeg, chunk), ce = ldc(a.chunk_cend, chunk);
  double lsum[RPL];
  int usum[RPL];
#pragma unroll
  for (int j = 0; j < RPL; ++j) { lsum[j] = 0.0; usum[j] = 0; }

  // the next clause's header is loaded while the current one is processed
  auto header = [&](int i, int* s, int* k) {
    const int t = __builtin_amdgcn_readfirstlane(a.clause_ids ? ldc(a.clause_ids, i) : i);
    *s = ldc(a.clause_ptr, t);
    *k = ldc(a.clause_ptr, t + 1) - *s;
  };
  int s_next = 0, k_next = 0;
  if (cb + wave < ce) header(cb + wave, &s_next, &k_next);
  for (int i = cb + wave; i < ce; i += WPB) {
    const int s = s_next, k = k_next;
    if (i + WPB < ce) header(i + WPB, &s_next, &k_next);
    const int m = (k + G - 1) / G;  // run length (the plan keeps m <= MAXC)
    const int lb = grp * m;         // first literal of this group's run
    float f[MAXC][RPL];
    int code[MAXC];
    int any_true[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) any_true[j] = 0;
    // gather the run: all its rows in flight together
#pragma clang loop unroll(full)
    for (int c = 0; c < MAXC; ++c) {
      const int li = lb + c;
      const bool in = c < m && li < k;
      code[c] = c < m ? ldc(a.clause_lits, s + (in ? li : 0)) : 0;
      float y[RPL];
      if (c < m) {
        // positions past the clause read its first literal's row again
        // and use factor 1
        load_row<RPL>(a.x + (int64_t)(code[c] >> 1) * a.ldx + rc, y);
      } else {
#pragma unroll
        for (int j = 0; j < RPL; ++j) y[j] = 0.0f;
      }
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        f[c][j] = in ? lit_factor(code[c], y[j]) : 1.0f;
        any_true[j] |= (in && lit_true(code[c], y[j])) ? 1 : 0;
      }
    }
#pragma unroll
    for (int j = 0; j < RPL; ++j) {
      // any literal true (per restart): OR over the groups
#pragma unroll
      for (int d = LPI; d < 64; d <<= 1) any_true[j] |= __shfl_xor(any_true[j], d);
    }
    // prefix within the run (exclusive), overwriting nothing: pre[c]
    float pre[MAXC][RPL];
    float run[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) run[j] = 1.0f;
#pragma clang loop unroll(full)
    for (int c = 0; c < MAXC; ++c) {
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        pre[c][j] = run[j];
        run[j] *= f[c][j];
      }
    }
    // products of the runs before (inclusive scan, then shift) and after
    float before[RPL], after[RPL], total[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) {
      float inc = run[j];
#pragma unroll
      for (int d = 1; d < G; d <<= 1) {
        const float o = __shfl_up(inc, d * LPI);
        inc = grp >= d ? inc * o : inc;
      }
      const float ex = __shfl_up(inc, LPI);
      before[j] = grp > 0 ? ex : 1.0f;
      total[j] = __shfl(inc, (G - 1) * LPI + lane);  // U_t: the product of all factors
      float sinc = run[j];
#pragma unroll
      for (int d = 1; d < G; d <<= 1) {
        const float o = __shfl_down(sinc, d * LPI);
        sinc = grp + d < G ? sinc * o : sinc;
      }
      const float sex = __shfl_down(sinc, LPI);
      after[j] = grp < G - 1 ? sex : 1.0f;
    }
    if (grp == 0) {
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        lsum[j] += (double)total[j];
        usum[j] += any_true[j] ? 0 : 1;
      }
    }
    // suffix within the run, then the partials
    float suf[RPL];
#pragma unroll
    for (int j = 0; j < RPL; ++j) suf[j] = after[j];
#pragma clang loop unroll(full)
    for (int c = MAXC - 1; c >= 0; --c) {
      float dv[RPL];
      const float slope = (code[c] & 1) ? 1.0f : -1.0f;
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        dv[j] = slope * ((before[j] * pre[c][j]) * suf[j]);
        suf[j] *= f[c][j];
      }
      const int li = lb + c;
      if (active && c < m && li < k)
        store_row<RPL>(a.D + (int64_t)ldc(a.lit_dslot, s + li) * a.ldD + r0, dv);
    }
  }
  block_partials<LPI, RPL>(lsum, usum, a.chunk_row ? ldc(a.chunk_row, chunk) : chunk, tile, a.R,
                           a.loss_part, a.unsat_part);
}

// ------------------------------------------------------------ finalize
//
// loss[f][r] = sum of the formula's partial rows (fixed order) + empty
// clauses; the same for the unsat count.
// RL lanes take neighbouring restarts (16 or 32 when there are no more), so
// a block of W waves has 64 W / RL row slots.  Slot q sums rows q, q + slots,
// ... in order, eight rows in flight; the slots' sums are then added pairwise
// in a fixed tree.
// STAGE kFinWhole: block x sums all rows of formula x.  Formulas of many
// rows take two launches: kFinParts cuts a formula's rows into a.split runs,
// one block each, written to part_l / part_u, and kFinJoin adds the parts.
// What bounds it: a block's trips are each one trip to memory (rows of other
// XCDs' writes), so rows per block are kept to about one trip.  684 rows of
// 500 restarts took 54 us in two parts of 64-lane rows, 18,842 rows of 16
// restarts 46 us.
enum { kFinWhole = 0, kFinParts = 1, kFinJoin = 2 };

template <int RL, int W, int STAGE>
__global__ __launch_bounds__(64 * W) void k_finalize(FinalizeArgs a) {
  constexpr int U = 8;
  constexpr int SL = 64 * W / RL;
  const int fl = STAGE == kFinParts ? blockIdx.x / a.split : blockIdx.x;
  const int f = a.f_base + fl;
  const int slot = threadIdx.x / RL, lane = threadIdx.x % RL;
  const int r = blockIdx.y * RL + lane;
  const int R = a.R;
  const double* lp = STAGE == kFinJoin ? a.part_l : a.loss_part;
  const int32_t* up = STAGE == kFinJoin ? a.part_u : a.unsat_part;
  int rb, re;
  if constexpr (STAGE == kFinJoin) {
    rb = fl * a.split;
    re = rb + a.split;
  } else {
    rb = a.a_beg[f];
    re = a.a_end[f];
    if constexpr (STAGE == kFinParts) {
      const int part = blockIdx.x % a.split, fb = rb, rows = re - rb;
      rb = fb + (int)((int64_t)rows * part / a.split);
      re = fb + (int)((int64_t)rows * (part + 1) / a.split);
    }
  }
  double acc = 0.0;
  int uacc = 0;
  if (r < R) {
    for (int row = rb + slot; row < re; row += U * SL) {
      double l[U];
      int c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) { l[u] = 0.0; c[u] = 0; }
      // rows past the end are read again in bounds and not added
      if (a.loss_out && !a.hard) {
#pragma unroll
        for (int u = 0; u < U; ++u) l[u] = lp[(int64_t)min(row + u * SL, re - 1) * R + r];
      }
      if (a.unsat_out || a.hard) {
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = up[(int64_t)min(row + u * SL, re - 1) * R + r];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool here = row + u * SL < re;
        acc += here ? l[u] : 0.0;
        uacc += here ? c[u] : 0;
      }
    }
  }
  __shared__ double sl[64 * W];
  __shared__ int su[64 * W];
  sl[threadIdx.x] = acc;
  su[threadIdx.x] = uacc;
  __syncthreads();
#pragma unroll
  for (int half = SL / 2; half >= 1; half /= 2) {
    if (slot < half) {
      sl[threadIdx.x] += sl[threadIdx.x + RL * half];
      su[threadIdx.x] += su[threadIdx.x + RL * half];
    }
    __syncthreads();
  }
  if (slot == 0 && r < R) {
    if constexpr (STAGE == kFinParts) {
      a.part_l[(int64_t)blockIdx.x * R + r] = sl[lane];
      a.part_u[(int64_t)blockIdx.x * R + r] = su[lane];
    } else {
      const int utot = su[lane] + a.n_empty[f];
      const double tot = a.hard ? (double)utot : sl[lane] + (double)a.n_empty[f];
      if (a.loss_out) a.loss_out[(int64_t)f * R + r] = (float)tot;
      if (a.unsat_out) a.unsat_out[(int64_t)f * R + r] = utot;
    }
  }
}

// ---------------------------------------------------------- init / copy

// Initial state: V restarts a lane (4 where the rows are 16 bytes apart), a
// wave of rows of LP lanes.  What bounds it: the VALU (four 64-bit products
// of the hash), and the writes; 123 M values took 308 us with a restart a
// lane and a thread per value.
template <int V>
__device__ __forceinline__ void init_row(float* x, uint64_t seed, int64_t v, int r) {
  float o[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const uint64_t key =
        ((uint64_t)(uint32_t)v << 32) + (uint64_t)(uint32_t)(r + e) + 0x9e3779b97f4a7c15ULL;
    const uint64_t h = splitmix_mix(seed ^ splitmix_mix(key));
    o[e] = (float)(h >> 40) * (1.0f / 16777216.0f);
  }
  store_row<V>(x, o);
}

// A thread's row within its workgroup and first column: LS (log2 of a row's
// lanes), or ls where LS is negative.  Shifts: a division by the number of
// lanes took as long as the draw of a value.
template <int V, int LS>
__device__ __forceinline__ void row_place(int32_t ls_arg, int* rows, int* sub, int* r) {
  const int ls = LS >= 0 ? LS : ls_arg;
  *rows = 256 >> ls;
  *sub = (int)threadIdx.x >> ls;
  *r = (((int)blockIdx.y << ls) + ((int)threadIdx.x & ((1 << ls) - 1))) * V;
}

template <int V, int LS>
__global__ __launch_bounds__(256) void k_init_state(float* __restrict__ x, int32_t ldx, int32_t n,
                                                    int32_t R, int32_t ls, uint64_t seed) {
  int rows, sub, r;
  row_place<V, LS>(ls, &rows, &sub, &r);
  if (r >= R) return;
  for (int64_t v = (int64_t)blockIdx.x * rows + sub; v < n; v += (int64_t)gridDim.x * rows)
    init_row<V>(x + v * ldx + r, seed, v, r);
}

// Copies.  Equal strides without padding columns: one run of 16-byte words
// (and a tail); else rows, four restarts a lane where both sides allow it.
__global__ __launch_bounds__(256) void k_copy_run(const float* __restrict__ src, float* __restrict__ dst,
                                                  int64_t count) {
  constexpr int U = 4;
  const int64_t words = count / 4, stride = (int64_t)gridDim.x * 256;
  const float4* s4 = reinterpret_cast<const float4*>(src);
  float4* d4 = reinterpret_cast<float4*>(dst);
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (; i + (U - 1) * stride < words; i += U * stride) {
    float4 t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = s4[i + u * stride];
#pragma unroll
    for (int u = 0; u < U; ++u) d4[i + u * stride] = t[u];
  }
  for (; i < words; i += stride) d4[i] = s4[i];
  if (blockIdx.x == 0 && threadIdx.x < count % 4)
    dst[words * 4 + threadIdx.x] = src[words * 4 + threadIdx.x];
}

template <int V, int LS>
__global__ __launch_bounds__(256) void k_copy_state(const float* __restrict__ src, int32_t lds,
                                                    float* __restrict__ dst, int32_t ldd, int32_t n,
                                                    int32_t R, int32_t ls) {
  constexpr int U = 4;
  int rows, sub, r;
  row_place<V, LS>(ls, &rows, &sub, &r);
  if (r >= R) return;
  const int64_t stride = (int64_t)gridDim.x * rows;
  for (int64_t v = (int64_t)blockIdx.x * rows + sub; v < n; v += U * stride) {
    float t[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v + u * stride < n) load_row<V>(src + (v + u * stride) * lds + r, t[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v + u * stride < n) store_row<V>(dst + (v + u * stride) * ldd + r, t[u]);
  }
}

__global__ void k_zero_i32(int32_t* p, int64_t count) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// ------------------------------------------------------- round & count
//
// bits[w][v]: bit l = [x[v][64w + l] > 0.5], 64-bit words, or one 32-bit word
// per variable when there are at most 32 restarts.

// Any state: P lanes per variable (P = 64, or 32 / 16 when all restarts fit
// one word and R <= P), so one ballot packs 64/P variables; a wave takes
// kPackU ballots' worth of consecutive variables per trip, all loads first.
constexpr int kPackU = 8;

template <int P, class Word>
__global__ __launch_bounds__(256) void k_pack_bits(const float* __restrict__ x, int32_t ldx, int32_t n,
                                                   int32_t R, Word* __restrict__ bits) {
  constexpr int VPB = 64 / P;  // variables per ballot
  const int wv = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int word = blockIdx.y;
  const int sub = lane / P, r = word * 64 + lane % P;
  for (int64_t v0 = ((int64_t)blockIdx.x * 4 + wv) * kPackU * VPB; v0 < n;
       v0 += (int64_t)gridDim.x * 4 * kPackU * VPB) {
    float val[kPackU];
#pragma unroll
    for (int u = 0; u < kPackU; ++u) {
      const int64_t v = v0 + u * VPB + sub;
      val[u] = (r < R && v < n) ? x[v * ldx + r] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kPackU; ++u) {
      const uint64_t m = __ballot(val[u] > 0.5f);
      const int64_t v = v0 + u * VPB + lane;  // lane k < VPB stores variable k's word
      if (lane < VPB && v < n) {
        uint64_t w = m;
        if constexpr (P < 64) w = (m >> (lane * P)) & ((1ULL << P) - 1ULL);
        bits[(int64_t)word * n + v] = (Word)w;
      }
    }
  }
}

// Rows of 16 bytes (R, ldx multiples of 4, x aligned): LP lanes take a word's
// restarts four at a time, their four bits are joined over 8 lanes (half of
// a 64-bit word) by DPP moves.  What bounds it: reading x; 123 M values took
// 158 us at 4 bytes a lane.
template <int LP, bool NARROW>
__global__ __launch_bounds__(256) void k_pack_rows(const float* __restrict__ x, int32_t ldx, int32_t n,
                                                   int32_t R, uint32_t* __restrict__ bits) {
  constexpr int VW = 64 / LP;  // variables of a wave's load
  constexpr int U = 8;
  const int wv = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int word = blockIdx.y, q = lane % LP, r = word * 64 + q * 4;
  for (int64_t v0 = ((int64_t)blockIdx.x * 4 + wv) * U * VW; v0 < n;
       v0 += (int64_t)gridDim.x * 4 * U * VW) {
    float val[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t v = v0 + u * VW + lane / LP;
      val[u][0] = val[u][1] = val[u][2] = val[u][3] = 0.0f;
      if (r < R && v < n) load_row<4>(x + v * ldx + r, val[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int m = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) m |= val[u][e] > 0.5f ? 1 << e : 0;
      m <<= 4 * (q % 8);
      m |= __builtin_amdgcn_update_dpp(0, m, 0xb1, 0xf, 0xf, false);   // lane ^ 1
      m |= __builtin_amdgcn_update_dpp(0, m, 0x4e, 0xf, 0xf, false);   // lane ^ 2
      if constexpr (LP > 4) m |= __builtin_amdgcn_update_dpp(0, m, 0x141, 0xf, 0xf, false);  // half row
      const int64_t v = v0 + u * VW + lane / LP;
      if (q % 8 == 0 && v < n) {
        if constexpr (NARROW) bits[v] = (uint32_t)m;
        else bits[((int64_t)word * n + v) * 2 + q / 8] = (uint32_t)m;
      }
    }
  }
}

// Lanes take one clause each; a clause's "unsatisfied" mask is the AND over
// its literals of "literal false", for all restarts of a word, and is added
// to the lane's bit-sliced counters.  These are emptied before they can
// overflow and at the end: 16 lanes' counters are added by DPP moves, then
// each lane reads its restarts' bits.
// LDS: the formula's words are copied to LDS first, so a literal costs an
// LDS read; without, its word comes from the L2.  Literals are read once.
// What bounds it: the VALU (about 9 operations a literal slot, trips of four,
// a wave's lanes as long as its longest clause).  384 formulas of up to
// 20,000 variables at 32 restarts: 304 us with 64-bit words from the L2 and
// a ballot and a popcount per restart and 64 clauses, 94 us with this; two
// or four clauses a lane in flight 100 us.
// A position past a clause's end reads its last literal again, which an AND
// does not notice.
template <int W, class Word, class Get>
__device__ __forceinline__ Word and_literals_false(const int32_t* lits, Get word_of, uint32_t p,
                                                   uint32_t last, Word mask) {
  int code[W];
  Word b[W];
#pragma unroll
  for (int u = 0; u < W; ++u) code[u] = lits[min(p + u, last)];
#pragma unroll
  for (int u = 0; u < W; ++u) b[u] = word_of((uint32_t)code[u] >> 1);
#pragma unroll
  for (int u = 0; u < W; ++u) mask &= ~(b[u] ^ (Word)((int64_t)(code[u] << 31) >> 31));
  return mask;
}

// planes += the planes of the lane a DPP move names; `p` planes are in use,
// the sum has one more.
template <int CTRL, int p, int TP, class Word>
__device__ __forceinline__ void add_dpp(Word (&c)[TP]) {
  Word carry = 0;
#pragma unroll
  for (int i = 0; i < p; ++i) {
    Word o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)c[i], CTRL, 0xf, 0xf, false);
    if constexpr (sizeof(Word) == 8)
      o |= (Word)(uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(c[i] >> 32), CTRL, 0xf, 0xf,
                                                       false)
           << 32;
    full_add<Word>(c[i], o, carry, c[i], carry);
  }
  c[p] = carry;
}

template <class Word, bool LDS, int T>
__global__ __launch_bounds__(T) void k_count_unsat(CountArgs a) {
  constexpr int B = 8 * sizeof(Word);
  constexpr int P = 5, TP = P + 4;  // planes of a lane, of 16 lanes' sum
  extern __shared__ int4 smem4[];
  Word* s_bits = reinterpret_cast<Word*>(smem4);
  __shared__ int s_cnt[B];
  const int tid = threadIdx.x, lane = tid & 63;
  const CountChunk ch = a.chunk[a.order[blockIdx.x]];
  const int word = blockIdx.y;
  const int rem = a.R - word * B;
  const Word valid = rem >= B ? ~(Word)0 : (((Word)1 << rem) - 1);
  const Word* bw = reinterpret_cast<const Word*>(a.bits) + (int64_t)word * a.n + ch.vb;
  if (tid < B) s_cnt[tid] = 0;
  if constexpr (LDS) {
    for (int i = tid; i < ch.nf; i += T) s_bits[i] = bw[i];
  }
  __syncthreads();
  auto word_of = [&](uint32_t v) -> Word {
    if constexpr (LDS) return s_bits[v - (uint32_t)ch.vb];
    else return bw[v - (uint32_t)ch.vb];
  };
  // positions relative to the run's first literal
  const int p0 = a.clause_ptr[ch.cb];
  const int32_t* lits = a.clause_lits + p0;
  Word c[P];
#pragma unroll
  for (int p = 0; p < P; ++p) c[p] = 0;
  auto empty = [&]() {
    Word all[TP];
#pragma unroll
    for (int p = 0; p < TP; ++p) all[p] = p < P ? c[p] : 0;
    add_dpp<0xb1, P>(all);       // lane ^ 1
    add_dpp<0x4e, P + 1>(all);   // lane ^ 2
    add_dpp<0x141, P + 2>(all);  // half rows mirrored
    add_dpp<0x140, P + 3>(all);  // rows mirrored: each lane its row's sum
#pragma unroll
    for (int r = lane % 16; r < B; r += 16) {
      int cnt = 0;
#pragma unroll
      for (int p = 0; p < TP; ++p) cnt += (int)(all[p] >> r & 1) << p;
      if (cnt) atomicAdd(&s_cnt[r], cnt);
    }
#pragma unroll
    for (int p = 0; p < P; ++p) c[p] = 0;
  };
  // a clause a lane and trip: its first four literals, then the rest (a
  // clause without literals stays unsatisfied)
  int room = (1 << P) - 1;
  for (int t = ch.cb + tid; __any(t < ch.ce); t += T) {
    const bool here = t < ch.ce;
    const uint32_t ps = here ? (uint32_t)(a.clause_ptr[t] - p0) : 0u;
    const uint32_t pe = here ? (uint32_t)(a.clause_ptr[t + 1] - p0) : 0u;
    Word mask = here ? valid : 0;
    uint32_t p = ps;
    for (; p + 16 <= pe; p += 8)  // long clauses
      mask = and_literals_false<8, Word>(lits, word_of, p, pe - 1, mask);
    for (; p < pe; p += 4)
      mask = and_literals_false<4, Word>(lits, word_of, p, pe - 1, mask);
    if (room == 0) {
      empty();
      room = (1 << P) - 1;
    }
    --room;
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const Word carry = c[p] & mask;
      c[p] ^= mask;
      mask = carry;
    }
  }
  empty();
  __syncthreads();
  const int r = word * B + tid;
  if (tid < B && r < a.R) a.unsat_part[(int64_t)a.order[blockIdx.x] * a.R + r] = s_cnt[tid];
}

// best[f] = argmin_r unsat[f][r], ties to the lowest r, via the packed key
// (unsat << 32) | r.
__global__ __launch_bounds__(256) void k_best(const int32_t* unsat, int32_t R, int32_t* best) {
  const int f = blockIdx.x;
  uint64_t key = ~0ULL;
  for (int r = threadIdx.x; r < R; r += 256) {
    const uint64_t k = ((uint64_t)(uint32_t)unsat[(int64_t)f * R + r] << 32) | (uint32_t)r;
    key = k < key ? k : key;
  }
  __shared__ uint64_t s[256];
  s[threadIdx.x] = key;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) s[threadIdx.x] = s[threadIdx.x + w] < s[threadIdx.x] ? s[threadIdx.x + w] : s[threadIdx.x];
    __syncthreads();
  }
  if (threadIdx.x == 0) best[f] = (int32_t)(s[0] & 0xffffffffULL);
}

template <class Word>
__global__ void k_best_assign(const Word* bits, int32_t n, const int32_t* var_formula,
                              const int32_t* best, uint8_t* out) {
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    const int r = best[var_formula[v]];
    constexpr int B = 8 * sizeof(Word);
    out[v] = (uint8_t)((bits[(int64_t)(r / B) * n + v] >> (r % B)) & 1);
  }
}

// ------------------------------------------------------------ launchers

namespace {

template <int LPI, int RPL>
hipError_t clause_pass_go(const ClausePassArgs& a, int, int chunks, int tiles, hipStream_t s) {
  hipLaunchKernelGGL((k_clause_pass<LPI, RPL>), dim3(chunks, tiles), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

// Clauses in flight a slot, and the exact tail, by the longest clause kmax.
// Many slots a workgroup (few lanes an item) hold a chunk's clauses in one
// trip, so more clauses a slot leave slots idle and put clauses one after
// another: 4,096 formulas of 16 to 64 variables at 16 restarts 35, 49 and 83 us
// with 1, 2 and 4 clauses (47 with the clause pass), Zipf of 100,000 at 16 132,
// 161 and 202, the formulas at 7 restarts 40, 38 and 47, 50,000 variables in
// 3-literal clauses at 128 restarts 56, 51 and 58.  With a wave a clause four
// hide each other's latency (50,000 at 333 restarts 218, 184 and 174), but not
// where clauses of many literals would follow each other in one slot (six of
// 5,000 literals at 512 restarts 668, 671 and 1,241).  The exact tail saves a
// wave up to three rows a clause (mixed lengths, 250,000 at 333 restarts 975
// us instead of 1,118) and costs formulas without a tail its branch (50,000 at
// 333 restarts 180 instead of 174).
template <int LPI, int RPL>
hipError_t loss_pass_go(const ClausePassArgs& a, int kmax, int chunks, int tiles, hipStream_t s) {
  const dim3 grid(chunks, tiles), block(kBlock);
  if constexpr (LPI == 64) {
    if (kmax <= 3) hipLaunchKernelGGL((k_loss_pass<LPI, RPL, 4, false>), grid, block, 0, s, a);
    else if (kmax <= 8) hipLaunchKernelGGL((k_loss_pass<LPI, RPL, 4, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_loss_pass<LPI, RPL, 2, true>), grid, block, 0, s, a);
  } else if constexpr (LPI == 32 && RPL == 4) {
    if (kmax <= 3) hipLaunchKernelGGL((k_loss_pass<LPI, RPL, 2, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_loss_pass<LPI, RPL, 2, true>), grid, block, 0, s, a);
  } else if constexpr (LPI == 4 || RPL == 4) {
    hipLaunchKernelGGL((k_loss_pass<LPI, RPL, 1, false>), grid, block, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_loss_pass<LPI, RPL, 2, false>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

#define GALSAT_TILE_RPL(GO, LPI)                                   \
  (t.rpl == 4   ? GO<LPI, 4>(a, kmax, chunks, tiles, s)            \
   : t.rpl == 2 ? GO<LPI, 2>(a, kmax, chunks, tiles, s)            \
                : GO<LPI, 1>(a, kmax, chunks, tiles, s))
#define GALSAT_TILES(GO)                                           \
  (t.lpi == 4    ? GALSAT_TILE_RPL(GO, 4)                          \
   : t.lpi == 8  ? GALSAT_TILE_RPL(GO, 8)                          \
   : t.lpi == 16 ? GALSAT_TILE_RPL(GO, 16)                         \
   : t.lpi == 32 ? GALSAT_TILE_RPL(GO, 32)                         \
                 : GALSAT_TILE_RPL(GO, 64))

hipError_t clause_tiles(const ClausePassArgs& a, Tile t, int chunks, int tiles, hipStream_t s) {
  const int kmax = 0;  // not used
  return GALSAT_TILES(clause_pass_go);
}

hipError_t loss_tiles(const ClausePassArgs& a, int kmax, Tile t, int chunks, int tiles, hipStream_t s) {
  return GALSAT_TILES(loss_pass_go);
}

#undef GALSAT_TILES
#undef GALSAT_TILE_RPL
}  // namespace

hipError_t launch_short_clause(const ClausePassArgs& a, Tile t, int ks, int chunks, hipStream_t s) {
  if (chunks <= 0) return hipSuccess;
  if (ks != 4 && ks != kShortClauseMax) return hipErrorInvalidValue;
  const int tiles = launch_tiles(a, t);
  dim3 grid(chunks, tiles), block(kBlock);
  switch (t.lpi * 8 + t.rpl) {
#define GALSAT_SHORT_CASE(L, P)                                                                 \
  case L * 8 + P:                                                                               \
    if (ks == 4)                                                                                \
      hipLaunchKernelGGL((k_short_clause<L, P, 4>), grid, block, 0, s, a);                      \
    else                                                                                        \
      hipLaunchKernelGGL((k_short_clause<L, P, kShortClauseMax>), grid, block, 0, s, a);        \
    break;
    GALSAT_SHORT_CASE(4, 1)
    GALSAT_SHORT_CASE(4, 2)
    GALSAT_SHORT_CASE(4, 4)
    GALSAT_SHORT_CASE(8, 1)
    GALSAT_SHORT_CASE(8, 2)
    GALSAT_SHORT_CASE(8, 4)
    GALSAT_SHORT_CASE(16, 1)
    GALSAT_SHORT_CASE(16, 2)
    GALSAT_SHORT_CASE(16, 4)
    GALSAT_SHORT_CASE(32, 1)
    GALSAT_SHORT_CASE(32, 2)
    GALSAT_SHORT_CASE(32, 4)
    GALSAT_SHORT_CASE(64, 1)
    GALSAT_SHORT_CASE(64, 2)
    GALSAT_SHORT_CASE(64, 4)
#undef GALSAT_SHORT_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_wave_clause(const ClausePassArgs& a, Tile t, int maxc, int chunks, hipStream_t s) {
  if (chunks <= 0) return hipSuccess;
  if (wave_clause_kmax(t) <= 0) return hipErrorInvalidValue;
  if (maxc != kWaveClauseSmallChunks && maxc != wave_clause_chunks(t.lpi)) return hipErrorInvalidValue;
  const int tiles = launch_tiles(a, t);
  dim3 grid(chunks, tiles), block(kBlock);
  switch (t.lpi * 8 + t.rpl) {
#define GALSAT_WAVE_CASE(L, P)                                                                  \
  case L * 8 + P:                                                                               \
    if (maxc == kWaveClauseSmallChunks)                                                         \
      hipLaunchKernelGGL((k_wave_clause<L, P, kWaveClauseSmallChunks>), grid, block, 0, s, a);  \
    else                                                                                        \
      hipLaunchKernelGGL((k_wave_clause<L, P, wave_clause_chunks(L)>), grid, block, 0, s, a);   \
    break;
    GALSAT_WAVE_CASE(4, 1)
    GALSAT_WAVE_CASE(4, 2)
    GALSAT_WAVE_CASE(4, 4)
    GALSAT_WAVE_CASE(8, 1)
    GALSAT_WAVE_CASE(8, 2)
    GALSAT_WAVE_CASE(8, 4)
    GALSAT_WAVE_CASE(16, 1)
    GALSAT_WAVE_CASE(16, 2)
    GALSAT_WAVE_CASE(16, 4)
#undef GALSAT_WAVE_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_clause_pass(const ClausePassArgs& a, Tile t, int chunks, hipStream_t s) {
  if (chunks <= 0) return hipSuccess;
  return clause_tiles(a, t, chunks, launch_tiles(a, t), s);
}

// own [m], ids [m], first [n + 1], cursor [n + 1]
size_t loss_list_scratch(int32_t m, int32_t n) { return 2 * (size_t)m + 2 * ((size_t)n + 1); }

hipError_t launch_loss_list(const int32_t* clause_ptr, const int32_t* clause_lits, int32_t m,
                            const int32_t* var_ptr, int32_t n, int32_t* tmp, int32_t* loss_ptr,
                            int32_t* loss_lits, hipStream_t s) {
  int32_t *own = tmp, *ids = own + m, *first = ids + m, *cursor = first + n + 1;
  const dim3 gm(grid_x_for(((int64_t)m + 256) / 256)), gn(grid_x_for(((int64_t)n + 255) / 256)), block(256);
  const hipError_t e = launch_zero_i32(first, 2 * ((int64_t)n + 1), s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_list_own, gm, block, 0, s, clause_ptr, clause_lits, m, var_ptr, n, own, first);
  hipLaunchKernelGGL(k_list_scan, dim3(1), dim3(1024), 0, s, first, (int64_t)n + 1);
  hipLaunchKernelGGL(k_list_place, gm, block, 0, s, own, m, first, cursor, ids);
  hipLaunchKernelGGL(k_list_order, gn, block, 0, s, first, cursor, n, ids);
  hipLaunchKernelGGL(k_list_lengths, gm, block, 0, s, clause_ptr, ids, m, loss_ptr);
  hipLaunchKernelGGL(k_list_scan, dim3(1), dim3(1024), 0, s, loss_ptr, (int64_t)m + 1);
  hipLaunchKernelGGL(k_list_copy, gm, block, 0, s, clause_ptr, clause_lits, ids, m, loss_ptr, loss_lits);
  return hipGetLastError();
}

hipError_t launch_loss_pass(const ClausePassArgs& a_in, int kmax, Tile t, int chunks, hipStream_t s) {
  if (chunks <= 0) return hipSuccess;
  ClausePassArgs a = a_in;
  const int tiles = launch_tiles(a, t);
  a.xcd_pin = a.xcd_pin && (tiles == 2 || tiles == 4 || tiles == 8) ? 1 : 0;
  return loss_tiles(a, kmax, t, chunks, tiles, s);
}

namespace {

template <int RL>
hipError_t finalize_rl(const FinalizeArgs& a_in, int F, hipStream_t s) {
  FinalizeArgs a = a_in;
  const int gy = (a.R + RL - 1) / RL;
  // one trip of a four-wave block; a formula of more rows than four trips of
  // sixteen waves, when the chip has room, is cut into such parts (a second
  // launch costs about what four trips do)
  constexpr int kTrip = 8 * 256 / RL;
  const int64_t blocks = (int64_t)F * gy;
  a.split = 1;
  if (a.part_l && a.part_u && a.max_rows > 16 * kTrip && blocks < 512) {
    const int64_t want = (a.max_rows + kTrip - 1) / kTrip;
    const int64_t fit = kFinalizeScratch / ((int64_t)F * a.R);
    const int64_t room = std::max<int64_t>(1, 2048 / blocks);
    a.split = (int)std::max<int64_t>(1, std::min(std::min(want, fit), room));
  }
  if (a.split > 1) {
    hipLaunchKernelGGL((k_finalize<RL, 4, kFinParts>), dim3(F * a.split, gy), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_finalize<RL, 16, kFinJoin>), dim3(F, gy), dim3(1024), 0, s, a);
  } else if (a.max_rows > kTrip) {
    hipLaunchKernelGGL((k_finalize<RL, 16, kFinWhole>), dim3(F, gy), dim3(1024), 0, s, a);
  } else {
    hipLaunchKernelGGL((k_finalize<RL, 4, kFinWhole>), dim3(F, gy), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_finalize(const FinalizeArgs& a, int F, hipStream_t s) {
  if (F <= 0) return hipSuccess;
  if (a.R <= 16) return finalize_rl<16>(a, F, s);
  if (a.R <= 32) return finalize_rl<32>(a, F, s);
  return finalize_rl<64>(a, F, s);
}

namespace {

// Log2 of the lanes of a row of R restarts, V a lane: up to 64 lanes.
int row_lanes_log2(int32_t R, int V) {
  int ls = 0;
  while (ls < 6 && (V << ls) < R) ++ls;
  return ls;
}

bool rows_of_16(const float* p, int32_t ld, int32_t R) {
  return R % 4 == 0 && ld % 4 == 0 && reinterpret_cast<uintptr_t>(p) % 16 == 0;
}

// Grid of a row kernel: rows / (256 / lanes) workgroups, or the chip several
// times over.
dim3 row_grid(int64_t n, int32_t R, int V, int ls, int64_t most) {
  const int64_t rows = 256 >> ls, gx = (n + rows - 1) / rows;
  const int32_t span = V << ls;
  return dim3((uint32_t)std::max<int64_t>(1, std::min(gx, most)), (R + span - 1) / span);
}

}  // namespace

hipError_t launch_init_state(float* x, int32_t ldx, int32_t n, int32_t R, uint64_t seed,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int V = rows_of_16(x, ldx, R) ? 4 : 1, ls = row_lanes_log2(R, V);
  const dim3 grid = row_grid(n, R, V, ls, 16384);
  if (V == 4) hipLaunchKernelGGL((k_init_state<4, -1>), grid, dim3(256), 0, s, x, ldx, n, R, ls, seed);
  else if (ls == 6) hipLaunchKernelGGL((k_init_state<1, 6>), grid, dim3(256), 0, s, x, ldx, n, R, ls, seed);
  else hipLaunchKernelGGL((k_init_state<1, -1>), grid, dim3(256), 0, s, x, ldx, n, R, ls, seed);
  return hipGetLastError();
}

hipError_t launch_copy_state(const float* src, int32_t lds, float* dst, int32_t ldd, int32_t n,
                             int32_t R, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const bool aligned = (reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % 16 == 0;
  if (lds == ldd && lds == R && aligned) {
    const int64_t count = (int64_t)n * R;
    const int64_t gx = std::max<int64_t>(1, std::min<int64_t>((count / 4 + 255) / 256, 8192));
    hipLaunchKernelGGL(k_copy_run, dim3((uint32_t)gx), dim3(256), 0, s, src, dst, count);
    return hipGetLastError();
  }
  const int V = rows_of_16(src, lds, R) && rows_of_16(dst, ldd, R) ? 4 : 1, ls = row_lanes_log2(R, V);
  const dim3 grid = row_grid(n, R, V, ls, 8192);
  if (V == 4) hipLaunchKernelGGL((k_copy_state<4, -1>), grid, dim3(256), 0, s, src, lds, dst, ldd, n, R, ls);
  else if (ls == 6) hipLaunchKernelGGL((k_copy_state<1, 6>), grid, dim3(256), 0, s, src, lds, dst, ldd, n, R, ls);
  else hipLaunchKernelGGL((k_copy_state<1, -1>), grid, dim3(256), 0, s, src, lds, dst, ldd, n, R, ls);
  return hipGetLastError();
}

hipError_t launch_zero_i32(int32_t* p, int64_t count, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_i32, dim3(grid_x_for((count + 255) / 256)), dim3(256), 0, s, p, count);
  return hipGetLastError();
}

hipError_t launch_pack_bits(const float* x, int32_t ldx, int32_t n, int32_t R, uint64_t* bits,
                            hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int words = (R + 63) / 64;
  uint32_t* narrow = reinterpret_cast<uint32_t*>(bits);
  if (R % 4 == 0 && ldx % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0) {
    const int lp = R <= 16 ? 4 : R <= 32 ? 8 : 16;
    const int64_t per_block = 4 * 8 * (64 / lp);
    dim3 grid(grid_x_for((n + per_block - 1) / per_block), words), block(256);
    if (lp == 4) hipLaunchKernelGGL((k_pack_rows<4, true>), grid, block, 0, s, x, ldx, n, R, narrow);
    else if (lp == 8) hipLaunchKernelGGL((k_pack_rows<8, true>), grid, block, 0, s, x, ldx, n, R, narrow);
    else hipLaunchKernelGGL((k_pack_rows<16, false>), grid, block, 0, s, x, ldx, n, R, narrow);
    return hipGetLastError();
  }
  const int P = R <= 16 ? 16 : R <= 32 ? 32 : 64;
  const int64_t per_block = 4 * kPackU * (64 / P);
  dim3 grid(grid_x_for((n + per_block - 1) / per_block), words), block(256);
  if (P == 16)
    hipLaunchKernelGGL((k_pack_bits<16, uint32_t>), grid, block, 0, s, x, ldx, n, R, narrow);
  else if (P == 32)
    hipLaunchKernelGGL((k_pack_bits<32, uint32_t>), grid, block, 0, s, x, ldx, n, R, narrow);
  else
    hipLaunchKernelGGL((k_pack_bits<64, uint64_t>), grid, block, 0, s, x, ldx, n, R, bits);
  return hipGetLastError();
}

namespace {

constexpr int kCountLdsMax = 128 << 10;  // bytes of a formula's words

template <class Word, bool LDS, int T>
hipError_t count_unsat_go(const CountArgs& a, int blocks, int32_t nf_max, hipStream_t s) {
  const size_t lds = LDS ? (size_t)nf_max * sizeof(Word) : 0;
  // the most that count_shape takes, as handles of other sizes may launch the
  // kernel from other threads
  if (lds > (size_t)(48 << 10)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_count_unsat<Word, LDS, T>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kCountLdsMax);
    if (e != hipSuccess) return e;
  }
  const dim3 grid(blocks, (a.R + 8 * (int)sizeof(Word) - 1) / (8 * (int)sizeof(Word)));
  hipLaunchKernelGGL((k_count_unsat<Word, LDS, T>), grid, dim3(T), lds, s, a);
  return hipGetLastError();
}

template <class Word>
hipError_t count_unsat_word(const CountArgs& a, int blocks, CountShape c, int32_t nf_max, hipStream_t s) {
  if (!c.lds) return count_unsat_go<Word, false, 256>(a, blocks, nf_max, s);
  return c.threads == 256 ? count_unsat_go<Word, true, 256>(a, blocks, nf_max, s)
                          : count_unsat_go<Word, true, 1024>(a, blocks, nf_max, s);
}

}  // namespace

// A formula's words in LDS while they leave room for one workgroup of 16
// waves a CU; above 32 KB a workgroup is that large, so the CU stays full.
CountShape count_shape(int32_t R, int32_t nf_max) {
  const int64_t bytes = (int64_t)nf_max * (R <= 32 ? 4 : 8);
  CountShape c;
  c.lds = bytes <= kCountLdsMax;
  c.threads = c.lds && bytes > (32 << 10) ? 1024 : 256;
  return c;
}

hipError_t launch_count_unsat(const CountArgs& a, int blocks, int32_t nf_max, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  const CountShape c = count_shape(a.R, nf_max);
  return a.R <= 32 ? count_unsat_word<uint32_t>(a, blocks, c, nf_max, s)
                   : count_unsat_word<uint64_t>(a, blocks, c, nf_max, s);
}

hipError_t launch_best(const int32_t* unsat, int32_t F, int32_t R, int32_t* best, hipStream_t s) {
  if (F <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_best, dim3(F), dim3(256), 0, s, unsat, R, best);
  return hipGetLastError();
}

hipError_t launch_best_assign(const uint64_t* bits, int32_t n, int32_t R, const int32_t* var_formula,
                              const int32_t* best, uint8_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const dim3 grid(grid_x_for(((int64_t)n + 255) / 256)), block(256);
  if (R <= 32)
    hipLaunchKernelGGL((k_best_assign<uint32_t>), grid, block, 0, s,
                       reinterpret_cast<const uint32_t*>(bits), n, var_formula, best, out);
  else
    hipLaunchKernelGGL((k_best_assign<uint64_t>), grid, block, 0, s, bits, n, var_formula, best, out);
  return hipGetLastError();
}

}  // namespace galsat
