// Small inputs (Section II): a call on a few thousand nodes is bound by its launches (about
// 5 us each on the device) and by each kernel's few dependent round trips, so these paths
// count into direct LDS tables and take one or two launches.
#pragma once

namespace cq {

// ---- scoring -------------------------------------------------------------------
// First launch: every workgroup holds all node labels in LDS, takes an equal share of the
// rows and counts its entries in an L x L table; column L of the table counts the rows'
// nodes.  Second launch: one workgroup adds the tables up and finishes the call.
// The tables are added in the workspace's slots: SS_WORDS(L) words per workgroup, the last
// one its label error flag.
// The finishing workgroup reads up to 32 tables of L x (L + 1) cells, so the line to member rows
// lies at a number of label ids: 16,384 nodes and 390,000 entries 39 us with 2 label ids (49 by
// member rows), 45 with 40 (45), 47 with 48 (45), 69 with 100 (42), 102 with 160 (42); 4,000
// nodes and 32,000 entries 28 with 2 (48), 36 with 48 (40).
constexpr int SS_MAX_N = 16384;   // nodes (32 KB of labels in LDS)
constexpr int SS_MAX_L = 48;      // label ids
constexpr int SS_MAX_WG = 32;
constexpr int SS_THREADS = 512;
constexpr int SS_UNROLL = 4;
__host__ __device__ constexpr int ss_cells(int L) { return L * (L + 1); }
__host__ __device__ constexpr int ss_words(int L) { return ss_cells(L) + 1; }
__host__ __device__ constexpr size_t ss_lds(int n, int L) { return 4 * (size_t)ss_cells(L) + 2 * (size_t)n; }

__global__ __launch_bounds__(SS_THREADS) void k_small_count(int n, const int32_t* __restrict__ labels,
                                                            const int32_t* __restrict__ perm, const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ col, int L, u32* __restrict__ slots) {
  extern __shared__ u32 s_tab[];
  __shared__ u32 s_ex[SS_THREADS];  // per wave: row starts among its rows' entries
  __shared__ u32 s_bad;
  const int cells = ss_cells(L);
  uint16_t* sl = reinterpret_cast<uint16_t*>(s_tab + cells);
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid == 0) s_bad = 0;
  for (int i = tid; i < cells; i += SS_THREADS) s_tab[i] = 0;
  u32 bad = 0;
  for (int u0 = tid; u0 < n; u0 += SS_THREADS * SS_UNROLL) {
    int c[SS_UNROLL];
#pragma unroll
    for (int k = 0; k < SS_UNROLL; ++k) {
      const int u = u0 + k * SS_THREADS;
      c[k] = u < n ? (perm ? perm[u] : u) : 0;
    }
#pragma unroll
    for (int k = 0; k < SS_UNROLL; ++k) c[k] = labels[c[k]];
#pragma unroll
    for (int k = 0; k < SS_UNROLL; ++k) {
      const int u = u0 + k * SS_THREADS;
      if (u >= n) continue;
      const bool ok = (u32)c[k] < (u32)L;
      bad |= !ok;
      sl[u] = ok ? (uint16_t)c[k] : (uint16_t)0;  // the result of a call with a label error is void
    }
  }
  __syncthreads();
  if (bad) s_bad = 1;
  const int r0 = (int)((long long)n * blockIdx.x / gridDim.x), r1 = (int)((long long)n * (blockIdx.x + 1) / gridDim.x);
  for (int r = r0 + tid; r < r1; r += SS_THREADS) atomicAdd(&s_tab[(u32)sl[r] * (L + 1) + L], 1u);
  constexpr int WAVES = SS_THREADS / 64;
  const int mc = min(64, max(4, (r1 - r0 + WAVES - 1) / WAVES));  // rows per wave and step
  u32* ex = s_ex + wv * 64;
  for (int m = r0 + wv * mc; m < r1; m += WAVES * mc) {
    const int rows = min(mc, r1 - m);
    const u32 e0 = (u32)rp[m], tot = (u32)rp[m + rows] - e0;
    ex[lane] = lane < rows ? (u32)rp[m + lane] - e0 : tot;  // no entry reaches the lanes past the rows
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (u32 eb = 0; eb < tot; eb += 64 * SS_UNROLL) {  // the wave stays converged
      u32 v[SS_UNROLL], a[SS_UNROLL];
#pragma unroll
      for (int k = 0; k < SS_UNROLL; ++k) v[k] = (u32)col[e0 + min(eb + lane + 64u * (u32)k, tot - 1u)];
#pragma unroll
      for (int k = 0; k < SS_UNROLL; ++k) {
        const u32 e = min(eb + lane + 64u * (u32)k, tot - 1u);
        u32 l = 0;  // last row with ex[l] <= e
#pragma unroll
        for (u32 s = 32; s > 0; s >>= 1)
          if (ex[l + s] <= e) l += s;
        a[k] = sl[m + l];
      }
#pragma unroll
      for (int k = 0; k < SS_UNROLL; ++k) {
        const u32 b = sl[v[k]];
        // neighbouring entries mostly join one community to itself
        (void)wave_count<1>(s_tab, a[k] * (L + 1) + b, eb + lane + 64u * (u32)k < tot);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  __syncthreads();
  u32* slot = slots + (size_t)blockIdx.x * ss_words(L);
  for (int i = tid; i < cells; i += SS_THREADS) slot[i] = s_tab[i];
  if (tid == 0) slot[cells] = s_bad;
}

// A community's penalty terms are added four labels at a time, as a thread of group_one adds
// the labels of one table word (at most 512 label ids: one word per thread there), so the
// bits are those of the other paths.
constexpr int SF_THREADS = 1024;
__global__ __launch_bounds__(SF_THREADS) void k_small_final(int L, int wgs, const u32* __restrict__ slots, ScoreVis vis,
                                                            long long n, long long twom, PerComm pc,
                                                            ScoreResultDev* __restrict__ out) {
  static_assert(SS_MAX_L <= 4 * 64 && SS_MAX_L <= 512, "one table word per lane");
  extern __shared__ u32 s_tab[];
  __shared__ u32 s_N[SS_MAX_L], s_D[SS_MAX_L], s_I[SS_MAX_L], s_NP[SS_MAX_L];
  __shared__ u64 s_PEN[2 * SS_MAX_L];
  __shared__ Ctl s_ctl;
  __shared__ ScorePart s_part;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int cells = ss_cells(L), words = ss_words(L);
  if (tid < (int)(sizeof(Ctl) / 4)) reinterpret_cast<u32*>(&s_ctl)[tid] = 0;
  __syncthreads();
  for (int i = tid; i < words; i += SF_THREADS) {
    u32 x[SS_MAX_WG], t = 0;
#pragma unroll
    for (int w = 0; w < SS_MAX_WG; ++w) x[w] = w < wgs ? slots[(size_t)w * words + i] : 0u;  // all loads in flight
#pragma unroll
    for (int w = 0; w < SS_MAX_WG; ++w) t += x[w];
    if (i < cells) {
      s_tab[i] = t;
      if (i % (L + 1) == L) s_N[i / (L + 1)] = t;
    } else if (t) {
      s_ctl.flags = F_LABEL;
    }
  }
  __syncthreads();
  vis.N = s_N;
  vis.I = s_I;
  vis.NP = s_NP;
  vis.PEN = s_PEN;
  vis.ctl = &s_ctl;
  for (int g = wv; g < L; g += SF_THREADS / 64) {  // one community per wave
    ScoreVis::State st;
    vis.begin_wave(st, (u32)g);
    u32 d = 0;
    const u32* row = s_tab + g * (L + 1);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = 4 * lane + k;
      const u32 x = j < L ? row[j] : 0u;
      d += x;
      if (x && j != g) vis.visit_n(st, (u32)j, x, s_N[j]);
    }
    vis.settle(st);
    const u32 deg = wave_sum_u32(d);
    if (lane == 0) {
      s_I[g] = row[g];
      s_D[g] = deg;
    }
    vis.finish_wave(st, (u32)g);
  }
  __syncthreads();
  score_final1_body(L, s_N, s_D, s_I, s_NP, s_PEN, (double)twom, pc, &s_part, 0, 1);
  if (tid == 0) score_metrics(s_part, n, twom, vis.ecap, &s_ctl, out, 0u);  // thread 0 wrote s_part
}

// ---- comparison ----------------------------------------------------------------
// One workgroup counts the contingency table in a direct LDS table and finishes the call.  The
// limits are what its LDS holds and what one workgroup reads faster than the bands' seven launches
// run: 300 nodes 28 to 40 us (61 to 75), 32,768 nodes 43 to 80 (88 to 154).
constexpr int SC_THREADS = 1024;
constexpr int SC_MAX_N = 32768;
constexpr int SC_MAX_L = 1024;      // label ids per side
constexpr int SC_MAX_CELLS = 28672; // La x Lb (112 KB)
constexpr int SC_UNROLL = 8;
__host__ __device__ constexpr size_t sc_lds(int La, int Lb) {
  return 4 * ((size_t)La * Lb + 2 * (size_t)La + 2 * (size_t)Lb) + 8 * ((size_t)La + 1);
}

__global__ __launch_bounds__(SC_THREADS) void k_small_compare(int n, const int32_t* __restrict__ la, int La,
                                                              const int32_t* __restrict__ lb, int Lb,
                                                              int32_t* __restrict__ eci, int32_t* __restrict__ ecj,
                                                              int64_t* __restrict__ ecnt, long long ecap,
                                                              CmpResultDev* __restrict__ out) {
  extern __shared__ __align__(8) u32 s_dyn_c[];
  u64* r_f = reinterpret_cast<u64*>(s_dyn_c);  // per row: largest F ratio (bits of a non-negative double)
  u32* s_cell = reinterpret_cast<u32*>(r_f + La);
  u32* s_a = s_cell + La * Lb;
  u32* r_max = s_a + La;
  u32* s_b = r_max + La;
  u32* c_max = s_b + Lb;
  __shared__ Ctl s_ctl;
  __shared__ u64 s_u[8][SC_THREADS / 64], s_x[6][SC_THREADS / 64];
  __shared__ double s_fs[SC_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int cells = La * Lb;
  for (int i = tid; i < cells + 2 * La + 2 * Lb; i += SC_THREADS) s_cell[i] = 0;
  for (int i = tid; i < La; i += SC_THREADS) r_f[i] = 0;
  if (tid < (int)(sizeof(Ctl) / 4)) reinterpret_cast<u32*>(&s_ctl)[tid] = 0;
  __syncthreads();
  u32 bad = 0;
  for (int u0 = 0; u0 < n; u0 += SC_THREADS * SC_UNROLL) {  // uniform trip count
    int a[SC_UNROLL], b[SC_UNROLL];
#pragma unroll
    for (int k = 0; k < SC_UNROLL; ++k) {
      const int u = u0 + tid + k * SC_THREADS;
      a[k] = u < n ? la[u] : 0;
      b[k] = u < n ? lb[u] : 0;
    }
#pragma unroll
    for (int k = 0; k < SC_UNROLL; ++k) {
      const bool in = u0 + tid + k * SC_THREADS < n;
      const bool ok = (u32)a[k] < (u32)La && (u32)b[k] < (u32)Lb;
      bad |= in && !ok;
      (void)wave_count<1>(s_cell, (u32)(a[k] * Lb + b[k]), in && ok);
      (void)wave_count<1>(s_a, (u32)a[k], in && ok);
      (void)wave_count<1>(s_b, (u32)b[k], in && ok);
    }
  }
  if (bad) s_ctl.flags = F_LABEL;
  __syncthreads();
  const double Nd = (double)n;
  u64 nz = 0, a11 = 0;
  Frac96Sum xl;
  for (int k = tid; k < cells; k += SC_THREADS) {
    const u32 x = s_cell[k];
    if (!x) continue;
    const int i = k / Lb, j = k - i * Lb;
    const double f = 2.0 * (double)x / (double)((u64)s_a[i] + (u64)s_b[j]);  // Eq. 3 ratio
    atomicMax(&r_f[i], (u64)__double_as_longlong(f));                        // f >= 0: the bits order as the values
    atomicMax(&r_max[i], x);
    atomicMax(&c_max[j], x);
    a11 += (u64)x * (u64)(x - 1u) / 2u;
    if (x > 1u) xl.add_wide((double)x / Nd * log((double)x));  // the cell's part of S (see CmpVis)
    nz += 1;
    if (ecap > 0) {
      const unsigned long long idx = atomicAdd(&s_ctl.export_count, 1ull);
      if ((long long)idx < ecap) {
        eci[idx] = i;
        ecj[idx] = j;
        ecnt[idx] = (int64_t)x;
      }
    }
  }
  // entropy terms beside the cells: rows from the last thread down, columns from the first up
  u64 Ka = 0, Kb = 0, X = 0, Y = 0, smax = 0;
  u128 sa = 0, sb = 0;
  for (int i = SC_THREADS - 1 - tid; i < La; i += SC_THREADS) {
    const u32 ai = s_a[i];
    if (ai == 0) continue;
    Ka += 1;
    X += (u64)ai * (u64)(ai - 1u) / 2u;
    sa += fix96((double)ai / Nd * log((double)ai));
  }
  for (int j = tid; j < Lb; j += SC_THREADS) {
    const u32 bj = s_b[j];
    if (bj == 0) continue;
    Kb += 1;
    Y += (u64)bj * (u64)(bj - 1u) / 2u;
    sb += fix96((double)bj / Nd * log((double)bj));
  }
  __syncthreads();
  double fsum = 0.0;
  for (int i = tid; i < La; i += SC_THREADS) {
    smax += r_max[i];
    fsum += (double)s_a[i] * __longlong_as_double((long long)r_f[i]);  // 0 for an empty row
  }
  for (int j = tid; j < Lb; j += SC_THREADS) smax += c_max[j];
  u64 u[8] = {Ka, Kb, a11, X, Y, smax, nz, 0};
  u128 x3[3] = {xl.value(), sa, sb};
#pragma unroll
  for (int k = 0; k < 7; ++k) u[k] = wave_sum_u64(u[k]);
#pragma unroll
  for (int k = 0; k < 3; ++k) x3[k] = wave_sum_u128(x3[k]);
  fsum = wave_sum_f64(fsum);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 7; ++k) s_u[k][wv] = u[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      s_x[2 * k][wv] = (u64)x3[k];
      s_x[2 * k + 1][wv] = (u64)(x3[k] >> 64);
    }
    s_fs[wv] = fsum;
  }
  __syncthreads();
  if (tid >= 64) return;
  // one wave: the waves' sums, then the metrics
  constexpr int NW = SC_THREADS / 64;
#pragma unroll
  for (int k = 0; k < 7; ++k) u[k] = wave_sum_u64(lane < NW ? s_u[k][lane] : 0ull);
#pragma unroll
  for (int k = 0; k < 3; ++k) x3[k] = wave_sum_u128(lane < NW ? ((u128)s_x[2 * k + 1][lane] << 64) | s_x[2 * k][lane] : (u128)0);
  if (lane == 0) {
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) t += s_fs[i];
    cmp_metrics(u[0], u[1], u[2], u[3], u[4], u[5], x3[0], x3[1], x3[2], t, u[6], n, ecap, &s_ctl, out);
  }
}

}  // namespace cq
