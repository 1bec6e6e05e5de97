// Tiles of a renumbered graph and the edge pass over them (Section II-B; Eqs. (8), (9)).
//
// The stored order puts most neighbours of a row near it; the rest (edges between
// communities, mostly) join random places.  Reading those neighbours' labels one by one is
// what an edge pass spends its time on: an L2 serves a random read per channel and cycle
// (265 G/s for the chip), and only if the labels fit it (77 G/s over 20 MB).  So the graph is
// also kept as tiles of TG_ROWS consecutive rows, and each tile's entries in two parts:
//   near  the neighbour lies in the tile's window of ids (TG_HALO before and after its rows):
//         16-bit offsets in the window, row by row;
//   far   all others, sorted by slice (TS_NODES consecutive ids) of the neighbour, then by
//         tile: the 16-bit place of the neighbour in its slice, and the row's number in its
//         tile (16 bits).
// A call takes two passes.  k_far_labels holds one slice's labels in LDS, walks the slice's far
// entries in order and writes their labels out in order: no random read leaves LDS.
// k_tile_gather then takes one tile per workgroup, with the window's labels in LDS: near
// entries read theirs there, far entries read consecutive words of the first pass.  Both
// passes stream: about 4 bytes per near entry and 8 per far entry, labels and staging aside.
//
// Measured on the 10M-node graph (199M entries, 30 % of them far): see k_tile_gather.
#pragma once

namespace cq {

constexpr int TG_THREADS = 1024;
constexpr int TG_ROWS = 1024;        // rows per tile, one per thread
constexpr int TG_HALO = 4096;        // ids of the window before and after the tile's rows
constexpr int TS_SHIFT = 15;
constexpr int TS_NODES = 1 << TS_SHIFT;  // ids per slice: 64 KB of 16-bit labels, 128 KB of 32-bit ones
constexpr int TG_MAX_SLICES = 512;   // n up to 2^24
static_assert(TG_ROWS == TG_THREADS, "one row per thread");
static_assert(TG_ROWS + 2 * TG_HALO <= 65536, "16-bit window offsets");

// First id of the window of the tile starting at row r0, and one past its last.
__host__ __device__ __forceinline__ int tile_w0(int r0) { return r0 > TG_HALO ? r0 - TG_HALO : 0; }
__host__ __device__ __forceinline__ int tile_w1(int r0, int n) {
  return n - r0 > TG_ROWS + TG_HALO ? r0 + TG_ROWS + TG_HALO : n;
}

// ---- load time -------------------------------------------------------------------
// One workgroup per tile: near entries per row (ncnt), far entries per slice
// (fcnt[slice * T + tile]).
__global__ __launch_bounds__(TG_THREADS) void k_tile_count(int n, int T, int S, const int32_t* __restrict__ rp,
                                                           const int32_t* __restrict__ col, u32* __restrict__ ncnt,
                                                           u32* __restrict__ fcnt) {
  __shared__ u32 s_far[TG_MAX_SLICES];
  __shared__ u32 s_near[TG_ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r0 = (int)blockIdx.x * TG_ROWS, rows = min(TG_ROWS, n - r0);
  const int w0 = tile_w0(r0), w1 = tile_w1(r0, n);
  for (int i = tid; i < S; i += TG_THREADS) s_far[i] = 0;
  s_near[tid] = 0;
  __syncthreads();
  for (int r = wv; r < rows; r += TG_THREADS / 64) {  // one wave per row
    const int a = rp[r0 + r], b = rp[r0 + r + 1];
    u32 near = 0;
    for (int e = a + lane; e < b; e += 64) {
      const int v = col[e];
      if (v >= w0 && v < w1) ++near;
      else atomicAdd(&s_far[v >> TS_SHIFT], 1u);
    }
    if (near) atomicAdd(&s_near[r], near);
  }
  __syncthreads();
  if (tid < rows) ncnt[r0 + tid] = s_near[tid];
  for (int i = tid; i < S; i += TG_THREADS) fcnt[(size_t)i * T + blockIdx.x] = s_far[i];
}

// fpt[tile * S + slice] = first far entry of (slice, tile) for tiles 0..T (T: the slice's end).
__global__ __launch_bounds__(256) void k_tile_table(int T, int S, const u32* __restrict__ fstart, u32* __restrict__ fpt) {
  const size_t total = ((size_t)T + 1) * S;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const size_t t = i / S, s = i - t * S;
    fpt[i] = fstart[s * T + t];  // the next slice's start ends this one
  }
}

// One workgroup per tile: writes its entries (and weights) to their places.
__global__ __launch_bounds__(TG_THREADS) void k_tile_place(int n, int T, int S, const int32_t* __restrict__ rp,
                                                           const int32_t* __restrict__ col, const float* __restrict__ w,
                                                           const u32* __restrict__ nrp, const u32* __restrict__ fpt,
                                                           uint16_t* __restrict__ ncol, float* __restrict__ nw,
                                                           uint16_t* __restrict__ fcol, uint16_t* __restrict__ frow,
                                                           float* __restrict__ fw) {
  __shared__ u32 s_far[TG_MAX_SLICES];
  __shared__ u32 s_near[TG_ROWS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r0 = (int)blockIdx.x * TG_ROWS, rows = min(TG_ROWS, n - r0);
  const int w0 = tile_w0(r0), w1 = tile_w1(r0, n);
  for (int i = tid; i < S; i += TG_THREADS) s_far[i] = fpt[(size_t)blockIdx.x * S + i];
  if (tid < rows) s_near[tid] = nrp[r0 + tid];
  __syncthreads();
  for (int r = wv; r < rows; r += TG_THREADS / 64) {
    const int a = rp[r0 + r], b = rp[r0 + r + 1];
    for (int e = a + lane; e < b; e += 64) {
      const int v = col[e];
      if (v >= w0 && v < w1) {
        const u32 at = atomicAdd(&s_near[r], 1u);
        ncol[at] = (uint16_t)(v - w0);
        if (w) nw[at] = w[e];
      } else {
        const u32 at = atomicAdd(&s_far[v >> TS_SHIFT], 1u);
        fcol[at] = (uint16_t)(v & (TS_NODES - 1));
        frow[at] = (uint16_t)r;
        if (w) fw[at] = w[e];
      }
    }
  }
}

// ---- pass 1 ------------------------------------------------------------------------
// Labels of the far entries in their order.  Workgroup (slice, part): the slice's labels in
// LDS, then its share of the slice's entries (first[slice] up to end[slice]), eight per
// thread and step.
constexpr int FL_THREADS = 1024;
template <class LT>
__global__ __launch_bounds__(FL_THREADS) void k_far_labels(int n, int parts, const u32* __restrict__ first,
                                                           const u32* __restrict__ end, const uint16_t* __restrict__ fcol, const LT* __restrict__ labx,
                                                           LT* __restrict__ fl) {
  extern __shared__ __align__(16) u32 s_slice[];
  const LT* lab = reinterpret_cast<const LT*>(s_slice);
  const int tid = threadIdx.x;
  const int slice = (int)blockIdx.x / parts, part = (int)blockIdx.x % parts;
  const u32 a = first[slice], b = end[slice];
  // parts cut at multiples of 8 entries; the first and last also take the unaligned ends
  const u32 v0 = (a + 7u) / 8u, v1 = max(v0, b / 8u);  // whole groups of 8 inside [a, b)
  const u32 per = (v1 - v0 + (u32)parts - 1u) / (u32)parts;
  const u32 g0 = min(v1, v0 + (u32)part * per), g1 = min(v1, g0 + per);
  const bool ends = part == 0;  // the few entries outside the whole groups
  if (g0 == g1 && !ends) return;
  {
    constexpr int PER = 16 / (int)sizeof(LT);
    const long long id0 = (long long)slice << TS_SHIFT;
    const int cnt = (int)min((long long)TS_NODES, (long long)n - id0);
    typedef u32 v4u __attribute__((ext_vector_type(4)));
    const v4u* src = reinterpret_cast<const v4u*>(labx + id0);  // 16-byte aligned; padded past n (workspace array)
    v4u* dst = reinterpret_cast<v4u*>(s_slice);
    for (int i = tid; i < (cnt + PER - 1) / PER; i += FL_THREADS) dst[i] = src[i];
  }
  __syncthreads();
  if (ends) {
    const u32 head = min(b, v0 * 8u), tail = max(head, v1 * 8u);
    if (tid < 8 && a + tid < head) fl[a + tid] = lab[fcol[a + tid]];
    if (tid >= 64 && tid < 72 && tail + (tid - 64) < b) fl[tail + (tid - 64)] = lab[fcol[tail + (tid - 64)]];
  }
  const uint4* src = reinterpret_cast<const uint4*>(fcol);
  for (u32 g = g0 + tid; g < g1; g += FL_THREADS) {
    const uint4 q = src[g];
    const u32 c4[4] = {q.x, q.y, q.z, q.w};
    u32 x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = (u32)lab[(c4[k >> 1] >> (16 * (k & 1))) & 0xFFFFu];
    if constexpr (sizeof(LT) == 2) {
      reinterpret_cast<uint4*>(fl)[g] = make_uint4(x[0] | x[1] << 16, x[2] | x[3] << 16, x[4] | x[5] << 16, x[6] | x[7] << 16);
    } else {
      reinterpret_cast<uint4*>(fl)[2 * (size_t)g] = make_uint4(x[0], x[1], x[2], x[3]);
      reinterpret_cast<uint4*>(fl)[2 * (size_t)g + 1] = make_uint4(x[4], x[5], x[6], x[7]);
    }
  }
}

// ---- pass 2 ------------------------------------------------------------------------
// One tile per workgroup, in one of two stagings (ctl->mode, chosen by k_colscan_rows).
//
// STAGE_BLOCKS: consecutive rows with the same label form a run.  An entry whose neighbour has
// the row's own label c only adds to 2|E_c^in| (and, weighted, its weight to 2 w_in(c)) and
// is not staged; the others are counted per run and kept in an LDS buffer, each run adds
// (own << 32) | others to community c's cursor with one atomic, which hands it consecutive
// places in the segment, and the buffer is written out there run by run.  When the buffer
// overflows (and for 32-bit labels) the tile's entries are walked a second time instead.
// Weighted: own-label weights are summed exactly per run and added to IWacc[c].
//
// STAGE_ROWS (a partition that does not follow the stored order, so that runs are hardly
// longer than a row): every entry goes to its row's place, start + chunk prefix + per-node
// offset, near entries first.
//
// Rows of near entries are found through s_row8, the row of every eighth entry, and a short
// walk.  Far entries come in one short run per slice: half-waves take a slice each.
constexpr int TG_CHUNK = 16384;               // near entries per step of the row table
constexpr int TG_BUF = 8192, TG_BUF_W = 4096; // entries of another label kept in LDS
constexpr int TG_UNROLL = 8;
template <class LT, bool WT>
struct TileLds {
  static constexpr int PER = 16 / (int)sizeof(LT);
  static constexpr int WIN = (TG_ROWS + 2 * TG_HALO + PER) / PER * 4;        // words of the label window
  static constexpr int BUF = sizeof(LT) == 2 ? (WT ? TG_BUF_W : TG_BUF) : 0; // (run << 16) | label
  static constexpr int WORDS = WIN + (TG_ROWS + 4) + TG_CHUNK / 16 + 4 * (TG_ROWS + 4) + BUF + (WT ? BUF + 4 * TG_ROWS : 0) +
                               2 * TG_MAX_SLICES;
  static constexpr size_t BYTES = 4 * (size_t)WORDS;
};

template <class LT, bool WT>
__global__ __launch_bounds__(TG_THREADS) void k_tile_gather(int n, int S, const int32_t* __restrict__ rp,
                                                            const u32* __restrict__ nrp, const uint16_t* __restrict__ ncol,
                                                            const u32* __restrict__ fpt, const uint16_t* __restrict__ frow,
                                                            const LT* __restrict__ fl, const LT* __restrict__ labx,
                                                            const u32* __restrict__ start, const u32* __restrict__ D,
                                                            unsigned long long* __restrict__ cur64, Ctl* __restrict__ ctl,
                                                            LT* __restrict__ CB, const float* __restrict__ nw,
                                                            const float* __restrict__ fw, float* __restrict__ CW,
                                                            unsigned long long* __restrict__ IWacc, int L, int chunk,
                                                            const u32* __restrict__ PM, const u32* __restrict__ loc) {
  using TL = TileLds<LT, WT>;
  constexpr u32 NOLAB = (u32)LabelT<LT>::SENTINEL;
  extern __shared__ __align__(16) u32 s_mem[];
  u32* s_win32 = s_mem;
  const LT* s_win = reinterpret_cast<const LT*>(s_win32);
  u32* s_nr = s_win32 + TL::WIN;                                       // near row starts (tile-relative)
  uint16_t* s_row8 = reinterpret_cast<uint16_t*>(s_nr + TG_ROWS + 4);  // row of every eighth near entry of a chunk
  u32* s_a = s_nr + TG_ROWS + 4 + TG_CHUNK / 16;  // blocks: run of every row;         rows: place of the row's first entry
  u32* s_b = s_a + TG_ROWS + 4;                   // blocks: first row of every run;   rows: next free place of the row's far entries
  u32* s_cnt = s_b + TG_ROWS + 4;                 // blocks: staged entries per run, then the next free place of the run
  u32* s_base = s_cnt + TG_ROWS + 4;              // blocks: place of the run's first staged entry
  u32* s_buf = s_base + TG_ROWS + 4;
  float* s_wbuf = reinterpret_cast<float*>(s_buf + TL::BUF);
  unsigned long long* s_ilo = reinterpret_cast<unsigned long long*>(s_buf + 2 * TL::BUF);  // WT: own-label weight sum per run
  unsigned long long* s_ihi = s_ilo + TG_ROWS;
  u32* s_seg = s_buf + TL::BUF + (WT ? TL::BUF + 4 * TG_ROWS : 0);  // far entries: first and end per slice
  __shared__ u32 s_wave[TG_THREADS / 64];
  __shared__ u32 s_nbuf;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = (n + TG_ROWS - 1) / TG_ROWS;
  // each XCD (workgroup b runs on XCD b % 8) takes a contiguous eighth of the tiles
  const int per = (T + 7) / 8, t = (int)(blockIdx.x % 8u) * per + (int)(blockIdx.x / 8u);
  if ((int)(blockIdx.x / 8u) >= per || t >= T) return;
  const bool by_rows = !WT && ctl->mode == STAGE_ROWS;
  const int r0 = t * TG_ROWS, rows = min(TG_ROWS, n - r0);
  const int w0 = tile_w0(r0), w1 = tile_w1(r0, n), roff = r0 - w0;
  const u32 nb = nrp[r0];
  const u32 ne = nrp[r0 + rows] - nb;
  {
    typedef u32 v4u __attribute__((ext_vector_type(4)));
    const v4u* src = reinterpret_cast<const v4u*>(labx + w0);  // w0 is a multiple of 1,024; the array is padded past n
    v4u* dst = reinterpret_cast<v4u*>(s_win32);
    for (int i = tid; i < (w1 - w0 + TL::PER - 1) / TL::PER; i += TG_THREADS) dst[i] = src[i];
    if (tid <= rows) s_nr[tid] = nrp[r0 + tid] - nb;
    if (tid == 0 && rows == TG_ROWS) s_nr[TG_ROWS] = ne;
    for (int i = tid; i < S; i += TG_THREADS) {
      s_seg[i] = fpt[(size_t)t * S + i];
      s_seg[S + i] = fpt[((size_t)t + 1) * S + i];
    }
    if (tid == 0) s_nbuf = 0;
  }
  __syncthreads();
  // Calls f(row, label, weight) for every entry of the tile (lanes of a wave on neighbouring
  // entries; f may use wave votes, which then see the calling lanes).  near_place: called
  // with the entry's number in its row too.
  auto for_near = [&](auto&& f) {
    for (u32 c0 = 0; c0 < ne; c0 += TG_CHUNK) {
      const u32 c1 = min(ne, c0 + (u32)TG_CHUNK);
      __syncthreads();  // the previous chunk's row table is no longer read
      if (tid < rows) {
        const u32 a = max(s_nr[tid], c0), b = min(s_nr[tid + 1], c1);
        for (u32 g = (a + 7u) / 8u; g * 8u < b; ++g) s_row8[g - c0 / 8u] = (uint16_t)tid;
      }
      __syncthreads();
      for (u32 eb = c0 + tid; eb < c1; eb += TG_THREADS * TG_UNROLL) {
        u32 off[TG_UNROLL], row[TG_UNROLL], x[TG_UNROLL];
        float wt[TG_UNROLL];
#pragma unroll
        for (int k = 0; k < TG_UNROLL; ++k) {
          const u32 e = min(eb + (u32)(k * TG_THREADS), c1 - 1u);  // in bounds; masked below
          off[k] = ncol[nb + e];
          wt[k] = WT ? nw[nb + e] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < TG_UNROLL; ++k) {
          const u32 e = min(eb + (u32)(k * TG_THREADS), c1 - 1u);
          u32 r = s_row8[(e - c0) >> 3];
          while (s_nr[r + 1] <= e) ++r;
          row[k] = r;
        }
#pragma unroll
        for (int k = 0; k < TG_UNROLL; ++k) x[k] = (u32)s_win[off[k]];
#pragma unroll
        for (int k = 0; k < TG_UNROLL; ++k) {
          const u32 e = eb + (u32)(k * TG_THREADS);
          if (e < c1) f(row[k], x[k], wt[k], e - s_nr[row[k]]);
        }
      }
    }
  };
  auto for_far = [&](auto&& f) {
    constexpr int HW = TG_THREADS / 32;
    const u32 hl = (u32)tid & 31u;
    for (int s = tid >> 5; s < S; s += 2 * HW) {  // two slices in flight
      const int s2 = s + HW < S ? s + HW : s;
      const u32 a = s_seg[s], b = s_seg[S + s];
      const u32 a2 = s_seg[s2], b2 = s2 != s ? s_seg[S + s2] : a2;
      const u32 len = max(b - a, b2 - a2);
      for (u32 i = hl; i < len; i += 32) {
        const bool in = a + i < b, in2 = a2 + i < b2;
        u32 r = 0, x = 0, r2 = 0, x2 = 0;
        float wa = 0.0f, wb = 0.0f;
        if (in) {
          r = frow[a + i];
          x = (u32)fl[a + i];
          if (WT) wa = fw[a + i];
        }
        if (in2) {
          r2 = frow[a2 + i];
          x2 = (u32)fl[a2 + i];
          if (WT) wb = fw[a2 + i];
        }
        if (in) f(r, x, wa);
        if (in2) f(r2, x2, wb);
      }
    }
  };
  if (by_rows) {
    if (tid < rows) {
      const int u = r0 + tid;
      const u32 c = (u32)s_win[roff + tid], lu = loc[u];
      u32 base = SENT;
      if (c != NOLAB && lu != SENT) base = start[c] + PM[(size_t)(u / chunk) * L + c] + lu;
      s_a[tid] = base;
      s_b[tid] = s_nr[tid + 1] - s_nr[tid];  // far entries follow the near ones
    }
    // (for_near's first barrier comes before the first use)
    for_near([&](u32 r, u32 x, float, u32 i) {
      const u32 base = s_a[r];
      if (base != SENT) CB[base + i] = (LT)x;
    });
    __syncthreads();  // a tile without near entries passes no barrier above
    for_far([&](u32 r, u32 x, float) {
      const u32 base = s_a[r];
      if (base != SENT) CB[base + atomicAdd(&s_b[r], 1u)] = (LT)x;
    });
    return;
  }
  // runs of rows with equal labels
  u32 nruns = 0;
  {
    const u32 c = tid < rows ? (u32)s_win[roff + tid] : 0u;
    const bool head = tid < rows && (tid == 0 || c != (u32)s_win[roff + tid - 1]);
    const u64 m = __ballot(head);
    if (lane == 0) s_wave[wv] = (u32)__popcll(m);
    __syncthreads();
    u32 before = 0;
#pragma unroll
    for (int i = 0; i < TG_THREADS / 64; ++i) {
      const u32 k = s_wave[i];
      if (i < wv) before += k;
      nruns += k;
    }
    const u32 run = before + (u32)__popcll(m & (~0ull >> (63 - lane))) - 1u;  // runs that start at or before this row
    if (tid < rows) s_a[tid] = run;
    if (head) s_b[run] = (u32)tid;
    if (tid == 0) s_b[nruns] = (u32)rows;
    if (tid < rows) {
      s_cnt[tid] = 0;
      if (WT) {
        s_ilo[tid] = 0ull;
        s_ihi[tid] = 0ull;
      }
    }
    __syncthreads();
  }
  // WT: a thread sums the own-label weights of its current run and adds them to the run's LDS
  // sum when the run changes (64-bit atomics, the low word's carry added to the high word)
  u32 wrun = SENT;
  WeightSum wacc;
  auto wflush = [&]() {
    if (wrun != SENT) {
      const unsigned long long old = atomicAdd(&s_ilo[wrun], (unsigned long long)wacc.lo);
      const unsigned long long hi = wacc.hi + (old + wacc.lo < old ? 1ull : 0ull);
      if (hi) atomicAdd(&s_ihi[wrun], hi);
    }
  };
  const u64 below = (1ull << lane) - 1ull;
  auto stage = [&](u32 r, u32 x, float w) {
    const u32 run = s_a[r];
    const bool inter = x != (u32)s_win[roff + r];
    if (WT && !inter) {
      if (run != wrun) {
        wflush();
        wrun = run;
        wacc = WeightSum();
      }
      u64 vlo, vhi;
      WeightSum::split(w, vlo, vhi);
      wacc.add(vlo, vhi);
    }
    const u64 m = __ballot(inter);
    if (m == 0) return;
    // slots once per wave, counts once per wave for the first lane's run
    const int lead = __ffsll((long long)m) - 1;
    const u32 rl = __shfl(run, lead, 64);
    const u64 ms = __ballot(inter && run == rl);
    u32 slot0 = 0;
    if (lane == lead) {
      slot0 = atomicAdd(&s_nbuf, (u32)__popcll(m));
      atomicAdd(&s_cnt[rl], (u32)__popcll(ms));
    }
    slot0 = __shfl(slot0, lead, 64);
    if (inter) {
      const u32 slot = slot0 + (u32)__popcll(m & below);
      if (slot < (u32)TL::BUF) {
        s_buf[slot] = (run << 16) | x;
        if (WT) s_wbuf[slot] = w;
      }
      if (run != rl) atomicAdd(&s_cnt[run], 1u);
    }
  };
  for_near([&](u32 r, u32 x, float w, u32) { stage(r, x, w); });
  for_far([&](u32 r, u32 x, float w) { stage(r, x, w); });
  if (WT) wflush();
  __syncthreads();
  // one claim per run
  if ((u32)tid < nruns) {
    const u32 ra = s_b[tid], rb = s_b[tid + 1];
    const u32 c = (u32)s_win[roff + ra];
    const u32 tot = (u32)(rp[r0 + rb] - rp[r0 + ra]), inter = s_cnt[tid];
    u32 base = SENT;
    if (c != NOLAB && tot > 0) {
      const unsigned long long old = atomicAdd(&cur64[c], ((unsigned long long)(tot - inter) << 32) | inter);
      const u32 lo = (u32)old;
      if (lo + inter <= D[c]) base = start[c] + lo;  // < 2^31, so never the SENT marker
      else atomicOr(&ctl->flags, F_SEGMENT);  // never expected: the tile's counts disagree with the degrees
      if (WT) {
        const unsigned long long ilo = s_ilo[tid], ihi = s_ihi[tid];
        if (ilo | ihi) {
          const unsigned long long was = atomicAdd(&IWacc[2 * (size_t)c], ilo);
          const unsigned long long h = ihi + (was + ilo < was ? 1ull : 0ull);
          if (h) atomicAdd(&IWacc[2 * (size_t)c + 1], h);
        }
      }
    }
    s_base[tid] = base;
    s_cnt[tid] = 0;
  }
  __syncthreads();
  const u32 nbuf = s_nbuf;
  if (nbuf <= (u32)TL::BUF) {
    // write the buffer out: each wave takes consecutive places per run (coalesced)
    for (u32 k = tid; k < nbuf; k += TG_THREADS) {
      const u32 ent = s_buf[k];
      const u32 run = ent >> 16;
      const u64 act = __ballot(true);
      const int lead = __ffsll((long long)act) - 1;
      const u32 rl = __shfl(run, lead, 64);
      const u64 ms = __ballot(run == rl);
      u32 p0 = 0;
      if (lane == lead) p0 = atomicAdd(&s_cnt[rl], (u32)__popcll(ms));
      p0 = __shfl(p0, lead, 64);
      const u32 rank = run == rl ? p0 + (u32)__popcll(ms & below) : atomicAdd(&s_cnt[run], 1u);
      const u32 base = s_base[run];
      if (base != SENT) {
        CB[base + rank] = (LT)(ent & 0xFFFFu);
        if (WT) CW[base + rank] = s_wbuf[k];
      }
    }
  } else {
    // buffer overflow (or 32-bit labels): walk the tile's entries again
    auto direct = [&](u32 r, u32 x, float w) {
      const u32 run = s_a[r], base = s_base[run];
      if (x != (u32)s_win[roff + r] && base != SENT) {
        const u32 rank = atomicAdd(&s_cnt[run], 1u);
        CB[base + rank] = (LT)x;
        if (WT) CW[base + rank] = w;
      }
    };
    for_near([&](u32 r, u32 x, float w, u32) { direct(r, x, w); });
    for_far([&](u32 r, u32 x, float w) { direct(r, x, w); });
  }
}

}  // namespace cq
