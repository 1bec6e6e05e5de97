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
constexpr int TG_MAX_SLICES = 4096;  // n up to 2^27 (12-bit slice numbers, 16 KB of counters at load time)
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
// is not staged; the others are counted per run, each run adds (own << 32) | others to
// community c's cursor with one atomic, which hands it consecutive places in the segment,
// and they are written there run by run.  Until then far entries stay in registers and near
// ones (few of them have another label) in an LDS buffer; what does not fit is read again.
// Weighted: own-label weights are summed exactly per run and added to IWacc[c].
//
// STAGE_ROWS (a partition that does not follow the stored order, so that runs are hardly
// longer than a row): every entry goes to its row's place, start + chunk prefix + per-node
// offset, near entries first.  The rows are put together in LDS and written from there by 16
// lanes each: written one by one, the far entries' 2-byte stores were one L2 request each
// (0.3 of 0.7 ms on the 10M-node graph).
//
// A tile is a chain of a few dependent loads, and two workgroups share a CU, so the pass is
// bound by latency and by LDS work per entry: a thread loads eight near entries at once and
// all of its far ones before the first is used, a wave's 512 near entries nearly always lie
// in one run (one LDS read per entry, two atomics per wave), and a far entry's slice is found
// through s_seg8, the slice of every eighth far entry, and a short walk.
constexpr int TG_FAR = 8;                     // far entries per thread held in registers
constexpr int TG_CHUNK = 16384;               // near entries per step of the row table (STAGE_ROWS)
constexpr int TG_BUF = 4096, TG_BUF_W = 1536; // near entries of another label kept in LDS
template <class LT, bool WT>
struct TileLds {
  static constexpr int PER = 16 / (int)sizeof(LT);
  static constexpr int WIN = (TG_ROWS + 2 * TG_HALO + PER) / PER * 4;        // words of the label window
  static constexpr int BUF = sizeof(LT) == 2 ? (WT ? TG_BUF_W : TG_BUF) : 0; // (run << 16) | label
  static constexpr int ARR = TG_ROWS + 4;
  static constexpr int BASE = WIN + 7 * ARR + BUF + (WT ? BUF + 4 * TG_ROWS : 0);
  static constexpr int seg(int S) { return 2 * (S + 2) + TG_FAR * TG_THREADS / 16; }  // the far entries' tables
  // 16-bit labels, unweighted: STAGE_ROWS puts the rows together in BUF and what follows it, so
  // the workgroup takes all that leaves room for two per CU
  static constexpr int FULL = ((80 << 10) - 640) / 4;
  static constexpr int words(int S) {
    return sizeof(LT) == 2 && !WT && BASE + seg(S) < FULL ? FULL : BASE + seg(S);
  }
  static constexpr size_t bytes(int S) { return 4 * (size_t)words(S); }
};
static_assert(TG_CHUNK / 16 + 2 <= TG_ROWS + 4, "the row table of STAGE_ROWS takes a row array");

template <class LT, bool WT>
__global__ __launch_bounds__(TG_THREADS, 8) void k_tile_gather(
    int n, int S, const int32_t* __restrict__ rp, const u32* __restrict__ nrp, const uint16_t* __restrict__ ncol,
    const u32* __restrict__ fpt, const uint16_t* __restrict__ frow, const LT* __restrict__ fl, const LT* __restrict__ labx,
    const u32* __restrict__ start, const u32* __restrict__ D, unsigned long long* __restrict__ cur64, Ctl* __restrict__ ctl,
    LT* __restrict__ CB, const float* __restrict__ nw, const float* __restrict__ fw, float* __restrict__ CW,
    unsigned long long* __restrict__ IWacc, int L, int chunk, const u32* __restrict__ PM, const u32* __restrict__ loc,
    int always_rows) {
  using TL = TileLds<LT, WT>;
  constexpr u32 NOLAB = (u32)LabelT<LT>::SENTINEL;
  constexpr int WAVES = TG_THREADS / 64;
  extern __shared__ __align__(16) u32 s_mem[];
  u32* s_win32 = s_mem;
  const LT* s_win = reinterpret_cast<const LT*>(s_win32);
  u32* s_nr = s_win32 + TL::WIN;   // near row starts (tile-relative); later the places of the runs
  u32* s_a = s_nr + TL::ARR;       // run (and 16-bit label) of every row
  u32* s_b = s_a + TL::ARR;        // first row of every run
  u32* s_cnt = s_b + TL::ARR;      // staged far entries per run (those in registers)
  u32* s_more = s_cnt + TL::ARR;   // the other staged entries per run, then the next free place after the former
  u32* s_base = s_more + TL::ARR;  // first near entry of every run
  u32* s_first = s_base + TL::ARR; // first stored entry of every run
  u32* s_place = s_nr;
  u32* s_buf = s_first + TL::ARR;
  float* s_wbuf = reinterpret_cast<float*>(s_buf + TL::BUF);
  unsigned long long* s_ilo = reinterpret_cast<unsigned long long*>(s_buf + 2 * TL::BUF);  // WT: own-label weight sum per run
  unsigned long long* s_ihi = s_ilo + TG_ROWS;
  u32* s_pre = s_mem + TL::words(S) - TL::seg(S);  // far entries before each slice
  u32* s_foff = s_pre + S + 2;                     // place of a slice's far entry j, minus j
  uint16_t* s_seg8 = reinterpret_cast<uint16_t*>(s_foff + S + 2);
  __shared__ u32 s_wave[WAVES];
  __shared__ u32 s_nbuf;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = (n + TG_ROWS - 1) / TG_ROWS;
  // each XCD (workgroup b runs on XCD b % 8) takes a contiguous eighth of the tiles
  const int per = (T + 7) / 8, t = (int)(blockIdx.x % 8u) * per + (int)(blockIdx.x / 8u);
  if ((int)(blockIdx.x / 8u) >= per || t >= T) return;
  const bool by_rows = !WT && sizeof(LT) == 2 && (always_rows || ctl->mode == STAGE_ROWS);  // see k_colscan_rows
  const int r0 = t * TG_ROWS, rows = min(TG_ROWS, n - r0);
  const int w0 = tile_w0(r0), w1 = tile_w1(r0, n), roff = r0 - w0;
  // Every load that depends on no other is issued first, then those that need the tile's first
  // near entry or the row's label; the LDS writes wait for all of them at once.
  constexpr int SPT = TG_MAX_SLICES / TG_THREADS;
  const int spt = (S + TG_THREADS - 1) / TG_THREADS;
  const int my_row = r0 + min(tid, rows - 1);
  typedef u32 v4u __attribute__((ext_vector_type(4)));
  constexpr int WV = TL::WIN / 4;                                // 16-byte words of the window
  constexpr int WPT = (WV + TG_THREADS - 1) / TG_THREADS;
  const int nwin = (w1 - w0 + TL::PER - 1) / TL::PER;
  const v4u* win = reinterpret_cast<const v4u*>(labx + w0);  // w0 is a multiple of 1,024; the array is padded past n
  v4u wreg[WPT];
#pragma unroll
  for (int i = 0; i < WPT; ++i) wreg[i] = win[min(tid + i * TG_THREADS, nwin - 1)];
  const u32 own = (u32)labx[my_row];
  const u32 row_n = nrp[my_row];
  const int row_e = rp[my_row];
  const u32 lu = by_rows ? loc[my_row] : 0u;
  // the thread's slices (consecutive): far entries [fa, fe) of each
  u32 fa[SPT], fe[SPT];
#pragma unroll
  for (int i = 0; i < SPT; ++i) {
    const int s = tid * spt + i;
    const bool in = i < spt && s < S;
    fa[i] = in ? fpt[(size_t)t * S + s] : 0u;
    fe[i] = in ? fpt[((size_t)t + 1) * S + s] : 0u;
  }
  const u32 nb = nrp[r0];
  const u32 ne = nrp[r0 + rows] - nb;
  const u32 ng = (nb & 7u) + ne;  // near entries from the 16-byte word that holds the first one
  const uint4* ncol8 = reinterpret_cast<const uint4*>(ncol + (nb & ~7u));
  // the wave's first block of near entries (word i holds entries 8 i .. 8 i + 7 from nb & ~7)
  uint4 ahead = make_uint4(0u, 0u, 0u, 0u);
  if ((u32)(8 * tid) < ng) ahead = ncol8[tid];
  // STAGE_ROWS: the row's place in its segment (SENT: not written, only with a label error,
  // which voids the result)
  u32 row_place = SENT;
  if (by_rows && own != NOLAB && lu != SENT) row_place = start[own] + PM[(size_t)(my_row / chunk) * L + own] + lu;
  {
    v4u* dst = reinterpret_cast<v4u*>(s_win32);
#pragma unroll
    for (int i = 0; i < WPT; ++i)
      if (tid + i * TG_THREADS < nwin) dst[tid + i * TG_THREADS] = wreg[i];
    if (tid < rows) s_nr[tid] = row_n - nb;
    if (tid == 0) {
      s_nr[rows] = ne;
      s_nbuf = 0;
    }
  }
  // far entries numbered slice by slice
  u32 nf = 0;
  {
    u32 cnt = 0;
#pragma unroll
    for (int i = 0; i < SPT; ++i) cnt += fe[i] - fa[i];
    const u32 incl = wave_incl_scan(cnt);
    if (lane == 63) s_wave[wv] = incl;
    __syncthreads();
    u32 pre = incl - cnt;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
      const u32 k = s_wave[i];
      if (i < wv) pre += k;
      nf += k;
    }
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      const int s = tid * spt + i;
      if (i >= spt || s >= S) break;
      const u32 c = fe[i] - fa[i];
      s_pre[s] = pre;
      s_foff[s] = fa[i] - pre;
      for (u32 g = (pre + 7u) / 8u; g * 8u < pre + c && g < (u32)(TG_FAR * TG_THREADS / 8); ++g) s_seg8[g] = (uint16_t)s;
      pre += c;
    }
    if (tid == 0) s_pre[S] = nf;
  }
  __syncthreads();
  // place of far entry j (slices without entries are walked over)
  auto far_at = [&](u32 j) {
    u32 s;
    if (j < (u32)(TG_FAR * TG_THREADS)) {
      s = s_seg8[j >> 3];
    } else {  // beyond the table: last slice whose entries start at or before j
      s = 0;
      for (u32 st = TG_MAX_SLICES / 2; st > 0; st >>= 1)
        if (s + st < (u32)S && s_pre[s + st] <= j) s += st;
    }
    while (s_pre[s + 1] <= j) ++s;
    return s_foff[s] + j;
  };
  // the thread's far entries j = tid + 1024 k: row << 16 | label (16-bit labels), all loads in flight
  u32 fat[TG_FAR], fr[TG_FAR], fx[TG_FAR];
#pragma unroll
  for (int k = 0; k < TG_FAR; ++k) {
    const u32 j = (u32)(tid + k * TG_THREADS);
    fr[k] = 0;
    fx[k] = 0;
    if (j < nf) {
      fat[k] = far_at(j);
      fr[k] = frow[fat[k]];
      fx[k] = (u32)fl[fat[k]];
    }
  }
  // Walks the tile's near entries in wave blocks of 512: f(e, off) with e the number of the
  // lane's first of eight entries (from nb & ~7) and off their window offsets, two per word.
  auto near_blocks = [&](auto&& f) {
    uint4 q = ahead;
    for (u32 b = (u32)wv * 512u; b < ng; b += WAVES * 512u) {
      const u32 next = b + WAVES * 512u + 8u * (u32)lane;
      uint4 q1 = make_uint4(0u, 0u, 0u, 0u);
      if (next < ng) q1 = ncol8[next / 8u];
      f(b, b + 8u * (u32)lane, q);
      q = q1;
    }
  };
  auto off_of = [](const uint4& q, int k) {
    const u32 w = k < 2 ? q.x : k < 4 ? q.y : k < 6 ? q.z : q.w;
    return (k & 1) ? w >> 16 : w & 0xFFFFu;
  };
  const u32 skip = nb & 7u;  // entry number of the tile's first near entry
  if (by_rows) {
    // Entries are placed relative to the tile's first entry, row by row.  Per row: end of its
    // near entries, and the place of near entry e minus e (one LDS read gives both); the next
    // free place of its far entries; the row's place in its segment.
    uint2* s_row = reinterpret_cast<uint2*>(s_a);  // s_a and s_b
    u32* s_far = s_cnt;
    uint16_t* s_row8 = reinterpret_cast<uint16_t*>(s_more);
    LT* s_out = reinterpret_cast<LT*>(s_buf);
    // entries put together in LDS (beyond: written straight away); the far tables' space too
    // once all far entries are in registers
    const u32 cap = ((u32)(s_pre - s_buf) + (nf <= (u32)(TG_FAR * TG_THREADS) ? (u32)TL::seg(S) : 0u)) * (4 / sizeof(LT));
    if (tid < rows) {
      const u32 a = s_nr[tid], b = s_nr[tid + 1], at = (u32)(row_e - rp[r0]);
      s_row[tid] = make_uint2(b + skip, at - a - skip);
      s_far[tid] = at + b - a;
      s_base[tid] = row_place;
    }
    auto put = [&](u32 r, u32 at, u32 x) {
      if (at < cap) s_out[at] = (LT)x;
      else if (s_base[r] != SENT) CB[s_base[r] + (at - (s_row[r].y + s_nr[r] + skip))] = (LT)x;
    };
    for (u32 c0 = 0; c0 < ng; c0 += TG_CHUNK) {
      const u32 c1 = min(ng, c0 + (u32)TG_CHUNK);
      __syncthreads();  // the far entries are in registers; the previous chunk's row table is no longer read
      if (tid < rows) {
        const u32 a = max(s_nr[tid] + skip, c0), b = min(s_nr[tid + 1] + skip, c1);
        const u32 lo = s_nr[tid] == 0 ? c0 : a;  // the first group starts before the tile's first entry
        if (a < b)
          for (u32 g = (lo + 7u) / 8u; g * 8u < b; ++g) s_row8[g - c0 / 8u] = (uint16_t)tid;
      }
      __syncthreads();
      for (u32 e0 = c0 + 8u * (u32)tid; e0 < c1; e0 += 8u * TG_THREADS) {
        const uint4 q = c0 == 0 && e0 == 8u * (u32)tid ? ahead : ncol8[e0 / 8u];
        u32 r = s_row8[(e0 - c0) / 8u];
        uint2 row = s_row[r];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const u32 e = e0 + (u32)k;
          if (e >= skip && e < c1) {
            while (row.x <= e) row = s_row[++r];
            put(r, row.y + e, (u32)s_win[off_of(q, k)]);
          }
        }
      }
    }
    __syncthreads();  // (a tile without near entries passes no barrier above)
#pragma unroll
    for (int k = 0; k < TG_FAR; ++k)
      if ((u32)(tid + k * TG_THREADS) < nf) put(fr[k], atomicAdd(&s_far[fr[k]], 1u), fx[k]);
    for (u32 j = (u32)(tid + TG_FAR * TG_THREADS); j < nf; j += TG_THREADS) {
      const u32 at = far_at(j), r = frow[at];
      put(r, atomicAdd(&s_far[r], 1u), (u32)fl[at]);
    }
    __syncthreads();
    for (int r = tid >> 4; r < rows; r += TG_THREADS / 16) {
      const u32 base = s_base[r], at = s_row[r].y + s_nr[r] + skip, end = min(s_far[r], cap);
      if (base == SENT) continue;
      for (u32 i = at + ((u32)tid & 15u); i < end; i += 16) CB[base + (i - at)] = s_out[i];
    }
    return;
  }
  // runs of rows with equal labels
  u32 nruns = 0;
  {
    const u32 c = own;
    const bool head = tid < rows && (tid == 0 || c != (u32)s_win[roff + tid - 1]);
    const u64 m = __ballot(head);
    if (lane == 0) s_wave[wv] = (u32)__popcll(m);
    __syncthreads();
    u32 before = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
      const u32 k = s_wave[i];
      if (i < wv) before += k;
      nruns += k;
    }
    const u32 run = before + (u32)__popcll(m & (~0ull >> (63 - lane))) - 1u;  // runs that start at or before this row
    if (tid < rows) s_a[tid] = sizeof(LT) == 2 ? (run << 16) | c : run;
    if (head) {
      s_b[run] = (u32)tid;
      s_first[run] = (u32)row_e;
      s_base[run] = s_nr[tid] + skip;
    }
    if (tid == 0) {
      s_b[nruns] = (u32)rows;
      s_first[nruns] = (u32)rp[r0 + rows];
    }
    if (tid < rows) {
      s_cnt[tid] = 0;
      s_more[tid] = 0;
      if (WT) {
        s_ilo[tid] = 0ull;
        s_ihi[tid] = 0ull;
      }
    }
    __syncthreads();
  }
  // run of near entry e: the last one whose rows' near entries start at or before e (runs
  // without near entries start where the next one does)
  u32 top = 0;
  if (nruns > 1) top = 1u << (31 - __clz((int)(nruns - 1)));
  auto run_of = [&](u32 e) {
    u32 l = 0;
    for (u32 st = top; st > 0; st >>= 1)
      if (l + st < nruns && s_base[l + st] <= e) l += st;
    return l;
  };
  auto label_of = [&](u32 run) { return (u32)s_win[roff + s_b[run]]; };
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
  auto own_weight = [&](u32 run, float w) {
    if (run != wrun) {
      wflush();
      wrun = run;
      wacc = WeightSum();
    }
    u64 vlo, vhi;
    WeightSum::split(w, vlo, vhi);
    wacc.add(vlo, vhi);
  };
  // calls f(k, run, own label) for the lane's near entries of block b that exist
  auto with_runs = [&](u32 b, u32 e0, auto&& f) {
    const u32 q0 = run_of(max(b, skip)), q1 = run_of(min(b + 512u, ng) - 1u);
    u32 run = q0;
    if (q0 != q1 && e0 < ng) run = run_of(max(e0, skip));
    u32 c = label_of(run);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const u32 e = e0 + (u32)k;
      if (e < skip || e >= ng) continue;
      if (q0 != q1 && run + 1 < nruns && s_base[run + 1] <= e) {
        do ++run;
        while (run + 1 < nruns && s_base[run + 1] <= e);
        c = label_of(run);
      }
      f(k, run, c);
    }
    return q0 == q1 ? q0 : SENT;
  };
  near_blocks([&](u32 b, u32 e0, const uint4& q) {
    u32 inter = 0;          // bit k: the lane's entry k has another label
    u32 rk[8];              // its run (blocks of several runs only)
    const u32 one = with_runs(b, e0, [&](int k, u32 run, u32 c) {
      const u32 x = (u32)s_win[off_of(q, k)];
      rk[k] = run;
      if (x != c) inter |= 1u << k;
      else if (WT) own_weight(run, nw[(nb & ~7u) + e0 + (u32)k]);
    });
    const u32 cnt = (u32)__popc(inter);
    const u32 incl = wave_incl_scan(cnt);
    const u32 total = (u32)__builtin_amdgcn_readlane((int)incl, 63);
    if (total == 0) return;
    u32 slot = 0;
    if (lane == 0) {
      slot = atomicAdd(&s_nbuf, total);
      if (one != SENT) atomicAdd(&s_more[one], total);
    }
    slot = (u32)__builtin_amdgcn_readfirstlane((int)slot) + incl - cnt;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (!((inter >> k) & 1u)) continue;
      if (one == SENT) atomicAdd(&s_more[rk[k]], 1u);
      if (slot < (u32)TL::BUF) {
        s_buf[slot] = (rk[k] << 16) | (u32)s_win[off_of(q, k)];
        if (WT) s_wbuf[slot] = nw[(nb & ~7u) + e0 + (u32)k];
      }
      ++slot;
    }
  });
  auto of_row = [&](u32 r, u32& run, u32& c) {
    const u32 q = s_a[r];
    run = sizeof(LT) == 2 ? q >> 16 : q;
    c = sizeof(LT) == 2 ? q & 0xFFFFu : (u32)s_win[roff + r];
  };
  // far entries: fr becomes the run (SENT: own label), and the entry's rank among the run's
  // staged entries is known at once
  u32 rank[TG_FAR];
#pragma unroll
  for (int k = 0; k < TG_FAR; ++k) {
    const bool in = (u32)(tid + k * TG_THREADS) < nf;
    u32 run = 0, c = 0;
    of_row(fr[k], run, c);  // row 0 where there is no entry
    const bool inter = in && fx[k] != c;
    if (WT && in && !inter) own_weight(run, fw[fat[k]]);
    fr[k] = inter ? run : SENT;
    rank[k] = wave_count<2>(s_cnt, run, inter);
  }
  for (u32 j = (u32)(tid + TG_FAR * TG_THREADS); j < nf; j += TG_THREADS) {
    const u32 at = far_at(j);
    u32 run, c;
    of_row(frow[at], run, c);
    if ((u32)fl[at] != c) atomicAdd(&s_more[run], 1u);
    else if (WT) own_weight(run, fw[at]);
  }
  if (WT) wflush();
  __syncthreads();
  // one claim per run
  if ((u32)tid < nruns) {
    const u32 ra = s_b[tid];
    const u32 c = (u32)s_win[roff + ra];
    const u32 tot = s_first[tid + 1] - s_first[tid], inter = s_cnt[tid] + s_more[tid];
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
    s_place[tid] = base;
    s_more[tid] = s_cnt[tid];
  }
  __syncthreads();
  auto put = [&](u32 run, u32 at, u32 x, float w) {
    const u32 base = s_place[run];
    if (base == SENT) return;
    CB[base + at] = (LT)x;
    if (WT) CW[base + at] = w;
  };
#pragma unroll
  for (int k = 0; k < TG_FAR; ++k)
    if (fr[k] != SENT) put(fr[k], rank[k], fx[k], WT ? fw[fat[k]] : 0.0f);
  for (u32 j = (u32)(tid + TG_FAR * TG_THREADS); j < nf; j += TG_THREADS) {
    const u32 at = far_at(j), x = (u32)fl[at];
    u32 run, c;
    of_row(frow[at], run, c);
    if (x != c) put(run, atomicAdd(&s_more[run], 1u), x, WT ? fw[at] : 0.0f);
  }
  const u32 nbuf = s_nbuf;
  if (nbuf <= (u32)TL::BUF) {
    // each wave takes consecutive places per run (coalesced)
    for (u32 k0 = 0; k0 < nbuf; k0 += TG_THREADS) {
      const u32 k = k0 + (u32)tid;
      const u32 ent = k < nbuf ? s_buf[k] : 0u;
      const u32 at = wave_count<2>(s_more, ent >> 16, k < nbuf);
      if (k < nbuf) put(ent >> 16, at, ent & 0xFFFFu, WT ? s_wbuf[k] : 0.0f);
    }
  } else {
    // more than the buffer holds (or 32-bit labels): walk the near entries again
    near_blocks([&](u32 b, u32 e0, const uint4& q) {
      (void)with_runs(b, e0, [&](int k, u32 run, u32 c) {
        const u32 x = (u32)s_win[off_of(q, k)];
        if (x != c) put(run, atomicAdd(&s_more[run], 1u), x, WT ? nw[(nb & ~7u) + e0 + (u32)k] : 0.0f);
      });
    });
  }
}

}  // namespace cq
