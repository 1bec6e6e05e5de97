// Tiles of a renumbered graph and the edge pass over them (Section II-B; Eqs. (8), (9)).
//
// The stored order puts most neighbours of a row near it; the rest (edges between
// communities, mostly) join random places.  Reading those neighbours' labels one by one is
// what an edge pass spends its time on: an L2 serves a random read per channel and cycle
// (265 G/s for the chip), and only if the labels fit it (77 G/s over 20 MB).  So the graph is
// also kept as tiles: the entries of TG_ROWS consecutive rows (a block of rows with many
// entries is cut into several tiles).  An entry is near when its neighbour lies in the block's
// window of ids (TG_HALO before and after its rows), else far.  Per graph:
//   eidx  one 16-bit word per entry, in row order: the place of the neighbour's label in the
//         tile's table, which holds the window's labels, then the tile's far labels;
//   fcol  the far entries sorted by chunk (consecutive tiles), slice (2^shift consecutive ids) of
//         the neighbour and tile: the 16-bit place of the neighbour in its slice;
//   fadr  for every tile, the numbers of its far entries in that order.
//
// A call takes two passes.  k_far_labels holds one slice's labels in LDS, walks the slice's far
// entries in order and writes their labels out in order: no random read leaves LDS.
// k_tile_gather then takes one tile per workgroup, puts its table together in LDS from the
// window and the far labels (one short run per slice), and finds every neighbour's label there.
// Both passes stream: 2 bytes per entry and 10 per far entry, labels and staging aside.
// A chunk has at most twice as many far entries as the graph has nodes (or one tile): a call whose
// workspace has no room for all far labels takes the two passes a few chunks at a time.
#pragma once

namespace cq {

constexpr int TG_THREADS = 1024;
constexpr int TG_WAVES = TG_THREADS / 64;
constexpr int TG_ROWS = 1024;        // rows per block, one per thread
constexpr int TG_HALO = 3584;        // ids of the window before and after the block's rows
constexpr int TG_WIN = TG_ROWS + 2 * TG_HALO;  // table places of the window (8,192); far labels follow
constexpr int TG_GROUP = 512;        // entries per wave and step: 8 per lane
constexpr int TG_STEPS = 3;          // steps per wave at most
constexpr int TG_ENT = TG_WAVES * TG_GROUP * TG_STEPS;  // entries per tile at most: 24,576
// A weighted graph's blocks with a tile of more far entries than this are cut into tiles of at
// most so many entries: two workgroups with 16-bit labels and the runs' weight sums still fit a
// CU's LDS then (a launch has the LDS of its largest tile).
// 10M nodes, 200M weighted entries: 601 us; with every block cut so 820, with column blocks 852.
constexpr int TG_ENT_W = 16384;
// Slices of 2^15 ids: 64 KB of 16-bit labels (two workgroups a CU), 128 KB of 32-bit ones.  Graphs
// whose tiles only ever serve 16-bit labels (more than 2^24 nodes) have slices of 2^16: a tile's
// far labels then are half as many, twice as long runs.  40M nodes: edge pass 1045 -> 934 us and
// far labels 141 -> 143; 10M nodes: 244 -> 238, but 52 -> 64.
constexpr int TS_SHIFT = 15;
constexpr int TS_SHIFT_LARGE = 16;
constexpr int TG_MAX_SLICES = 2048;  // n up to 2^27 (16 KB of counters at load time)
static_assert(TG_ROWS == TG_THREADS, "one row per thread");
static_assert(2 * (TG_WIN + TG_ENT) <= 65536, "16-bit table places, in units of 2 bytes");

struct Tile {
  int b0;       // first row of its block
  int r0, r1;   // rows with entries in the tile
  u32 e0, ne;   // first stored entry, entries
  u32 g0;       // first group of eidx
  u32 f0, nf;   // first word of fadr, far entries
};

// First id of the window of the block starting at row b0, and one past its last.
__host__ __device__ __forceinline__ int tile_w0(int b0) { return b0 > TG_HALO ? b0 - TG_HALO : 0; }
__host__ __device__ __forceinline__ int tile_w1(int b0, int n) {
  return n - b0 > TG_ROWS + TG_HALO ? b0 + TG_ROWS + TG_HALO : n;
}
// Place of a tile's entry i in eidx, from the tile's first word: a lane's 16-byte word holds
// entries 64 apart, so that a wave's k-th entries are consecutive.
__device__ __forceinline__ u32 tile_word(u32 i) {
  return (i & ~(u32)(TG_GROUP - 1)) + (i & 63u) * 8u + ((i >> 6) & 7u);
}

// ---- load time -------------------------------------------------------------------
// Tiles per block of rows (at least one), and the tiles themselves once their numbers are known;
// a tile of block b has at most ents[b] entries (no ents: TG_ENT).
__global__ __launch_bounds__(256) void k_tile_blocks(int n, int blocks, const u32* __restrict__ ents, const int32_t* __restrict__ rp,
                                                     u32* __restrict__ cnt) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= blocks) return;
  const u32 ent = ents ? ents[b] : (u32)TG_ENT;
  const u32 ne = (u32)(rp[min(n, (b + 1) * TG_ROWS)] - rp[b * TG_ROWS]);
  cnt[b] = max(1u, (ne + ent - 1u) / ent);
}

__global__ __launch_bounds__(256) void k_tile_list(int n, int blocks, const u32* __restrict__ ents, const int32_t* __restrict__ rp,
                                                   const u32* __restrict__ first, Tile* __restrict__ tiles,
                                                   u32* __restrict__ groups) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= blocks) return;
  const u32 ent = ents ? ents[b] : (u32)TG_ENT;
  const int b0 = b * TG_ROWS, b1 = min(n, b0 + TG_ROWS);
  const u32 E0 = (u32)rp[b0], E1 = (u32)rp[b1];
  for (u32 t = first[b], k = 0; t < first[b + 1]; ++t, ++k) {
    const u32 a = E0 + k * ent, z = min(E1, a + ent);
    // rows [r0, r1): all rows of the block for a single tile, else those with entries in [a, z)
    int r0 = b0, r1 = b1;
    if (first[b + 1] - first[b] > 1) {
      int lo = b0, hi = b1 - 1;  // last row starting at or before a
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if ((u32)rp[mid] <= a) lo = mid; else hi = mid - 1;
      }
      r0 = lo;
      hi = b1 - 1;  // last row starting before z
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if ((u32)rp[mid] < z) lo = mid; else hi = mid - 1;
      }
      r1 = lo + 1;
    }
    tiles[t] = Tile{b0, r0, r1, a, z - a, 0u, 0u, 0u};
    groups[t] = (z - a + TG_GROUP - 1u) / TG_GROUP;
  }
}

// ents[b] for tiles cut without it, whose far entries are counted in nfar.
__global__ __launch_bounds__(256) void k_tile_ents(int blocks, const u32* __restrict__ first, const u32* __restrict__ nfar,
                                                   u32 limit, u32* __restrict__ ents) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  if (b >= blocks) return;
  u32 most = 0;
  for (u32 t = first[b]; t < first[b + 1]; ++t) most = max(most, nfar[t]);
  ents[b] = most > limit ? (u32)TG_ENT_W : (u32)TG_ENT;
}

// The chunks of tiles: chunk c is tiles [first[c], first[c + 1]), of[t] tile t's chunk.
struct TileChunks {
  const u32* first;
  const u32* of;
  // tile t's place among the counters by chunk, slice and tile: at(t, s) = base + s * stride
  __device__ __forceinline__ void at(u32 t, int S, size_t& base, u32& stride) const {
    const u32 c = of[t], a = first[c];
    stride = first[c + 1] - a;
    base = (size_t)a * (u32)S + (t - a);
  }
};

// One workgroup per tile: far entries per slice (fcnt, by chunk, slice and tile; or null: the
// chunks are not known yet), in all, and the most of any tile.
__global__ __launch_bounds__(TG_THREADS) void k_tile_count(int n, int S, int shift, const Tile* __restrict__ tiles,
                                                           const int32_t* __restrict__ col, TileChunks chunks,
                                                           u32* __restrict__ fcnt, u32* __restrict__ nfar,
                                                           u32* __restrict__ fmax) {
  __shared__ u32 s_far[TG_MAX_SLICES];
  __shared__ u32 s_all;
  const Tile t = tiles[blockIdx.x];
  const int w0 = tile_w0(t.b0), w1 = tile_w1(t.b0, n);
  for (int i = threadIdx.x; i < S; i += TG_THREADS) s_far[i] = 0;
  if (threadIdx.x == 0) s_all = 0;
  __syncthreads();
  u32 mine = 0;
  for (u32 i = threadIdx.x; i < t.ne; i += TG_THREADS) {
    const int v = col[t.e0 + i];
    if (v >= w0 && v < w1) continue;
    ++mine;
    atomicAdd(&s_far[v >> shift], 1u);
  }
  if (mine) atomicAdd(&s_all, mine);
  __syncthreads();
  if (fcnt) {
    size_t base;
    u32 stride;
    chunks.at(blockIdx.x, S, base, stride);
    for (int i = threadIdx.x; i < S; i += TG_THREADS) fcnt[base + (size_t)i * stride] = s_far[i];
  } else if (threadIdx.x == 0) {
    nfar[blockIdx.x] = s_all;
    atomicMax(fmax, s_all);
  }
}

// out[chunk * S + slice] = their first far entry (after the last: the number of far entries).
__global__ __launch_bounds__(256) void k_tile_slices(int C, int S, const u32* __restrict__ first, const u32* __restrict__ fstart,
                                                     u32* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i > C * S) return;
  const int c = i / S, s = i % S;
  const u32 a = first[c];
  out[i] = fstart[(size_t)a * (u32)S + (c < C ? (size_t)s * (first[c + 1] - a) : 0)];
}

// One workgroup per tile: writes its entries' table places and its far entries.
__global__ __launch_bounds__(TG_THREADS) void k_tile_place(int n, int S, int shift, Tile* __restrict__ tiles,
                                                           const u32* __restrict__ group0, const u32* __restrict__ far0,
                                                           const int32_t* __restrict__ col, const u32* __restrict__ fcnt,
                                                           const u32* __restrict__ fstart, TileChunks chunks,
                                                           uint16_t* __restrict__ eidx, uint16_t* __restrict__ fcol,
                                                           u32* __restrict__ fadr) {
  __shared__ u32 s_pre[TG_MAX_SLICES];  // far entries of the tile before the slice
  __shared__ u32 s_cnt[TG_MAX_SLICES];
  const int tid = threadIdx.x;
  const Tile t = tiles[blockIdx.x];
  const int w0 = tile_w0(t.b0), w1 = tile_w1(t.b0, n);
  size_t base;
  u32 stride;
  chunks.at(blockIdx.x, S, base, stride);
  for (int i = tid; i < S; i += TG_THREADS) {
    s_pre[i] = fcnt[base + (size_t)i * stride];
    s_cnt[i] = 0;
  }
  __syncthreads();
  if (tid == 0) {
    u32 run = 0;
    for (int i = 0; i < S; ++i) {
      const u32 c = s_pre[i];
      s_pre[i] = run;
      run += c;
    }
  }
  __syncthreads();
  const u32 g0 = group0[blockIdx.x], f0 = far0[blockIdx.x];
  uint16_t* out = eidx + (size_t)g0 * TG_GROUP;
  for (u32 i = tid; i < t.ne; i += TG_THREADS) {
    const int v = col[t.e0 + i];
    u32 at = (u32)(v - w0);
    if (v < w0 || v >= w1) {
      const int s = v >> shift;
      const u32 k = atomicAdd(&s_cnt[s], 1u), j = s_pre[s] + k, g = fstart[base + (size_t)s * stride] + k;
      fcol[g] = (uint16_t)(v & ((1 << shift) - 1));
      fadr[f0 + j] = g;
      at = (u32)TG_WIN + j;
    }
    out[tile_word(i)] = (uint16_t)(2u * at);
  }
  if (tid == 0) {
    tiles[blockIdx.x].g0 = g0;
    tiles[blockIdx.x].f0 = f0;
    tiles[blockIdx.x].nf = far0[blockIdx.x + 1] - f0;
  }
}

// ---- pass 1 ------------------------------------------------------------------------
// Labels of the far entries of chunks [c0, c1) in their order.  Workgroup (slice, part): the
// slice's labels in LDS, then its share of the slice's entries, eight per thread and step: some
// of the chunks, or (parts >= chunks) one of parts / chunks shares of a chunk.  Returns at once
// when the gate's mode is STAGE_ROWS.
constexpr int FL_THREADS = 1024;
template <class LT>
__global__ __launch_bounds__(FL_THREADS) void k_far_labels(int n, int shift, int S, int c0, int c1, int parts,
                                                           const u32* __restrict__ first, const uint16_t* __restrict__ fcol,
                                                           const LT* __restrict__ labx, LT* __restrict__ fl,
                                                           const Ctl* __restrict__ gate) {
  extern __shared__ __align__(16) u32 s_slice[];
  const LT* lab = reinterpret_cast<const LT*>(s_slice);
  if (gate && gate->mode == STAGE_ROWS) return;
  const int tid = threadIdx.x;
  const int slice = (int)blockIdx.x / parts, part = (int)blockIdx.x % parts;
  const int nc = c1 - c0, sub = parts >= nc ? parts / nc : 1;  // parts = nc * sub, or fewer than nc
  const int ca = parts >= nc ? c0 + part / sub : c0 + (int)((long long)part * nc / parts);
  const int cb = parts >= nc ? ca + 1 : c0 + (int)((long long)(part + 1) * nc / parts);
  const u32 share = parts >= nc ? (u32)(part % sub) : 0u;
  {
    constexpr int PER = 16 / (int)sizeof(LT);
    const long long id0 = (long long)slice << shift;
    const int cnt = (int)min(1ll << shift, (long long)n - id0);
    typedef u32 v4u __attribute__((ext_vector_type(4)));
    const v4u* src = reinterpret_cast<const v4u*>(labx + id0);  // 16-byte aligned; padded past n (workspace array)
    v4u* dst = reinterpret_cast<v4u*>(s_slice);
    for (int i = tid; i < (cnt + PER - 1) / PER; i += FL_THREADS) dst[i] = src[i];
  }
  __syncthreads();
  u32 turn = 0;  // the thread that takes the next group of 8: every wave gets its share of all chunks together
  for (int c = ca; c < cb; ++c) {
    const u32 a = first[(size_t)c * S + slice], b = first[(size_t)c * S + slice + 1];
    // shares cut at multiples of 8 entries; the first share also takes the unaligned ends
    const u32 v0 = (a + 7u) / 8u, v1 = max(v0, b / 8u);  // whole groups of 8 inside [a, b)
    const u32 per = (v1 - v0 + (u32)sub - 1u) / (u32)sub;
    const u32 g0 = min(v1, v0 + share * per), g1 = min(v1, g0 + per);
    if (share == 0) {
      const u32 head = min(b, v0 * 8u), tail = max(head, v1 * 8u);
      if (tid < 8 && a + tid < head) fl[a + tid] = lab[fcol[a + tid]];
      if (tid >= 64 && tid < 72 && tail + (tid - 64) < b) fl[tail + (tid - 64)] = lab[fcol[tail + (tid - 64)]];
    }
    const uint4* src = reinterpret_cast<const uint4*>(fcol);
    for (u32 g = g0 + (((u32)tid - turn) & (FL_THREADS - 1u)); g < g1; g += FL_THREADS) {
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
    turn = (turn + (g1 - g0)) & (FL_THREADS - 1u);
  }
}

// ---- pass 2 ------------------------------------------------------------------------
// One tile per workgroup (T tiles from t0 on), in one of two stagings (ctl->mode, chosen by
// k_colscan_rows; rows = TG_BY_ROWS: by rows in any case; TG_RUNS_ONLY: nothing is done when the
// mode is STAGE_ROWS).
//
// STAGE_BLOCKS: consecutive rows (with entries) of the same label form a run.  An entry whose
// neighbour has the row's own label c only adds to 2|E_c^in| (and, weighted, its weight to
// 2 w_in(c)) and is not staged.  The others are numbered through the tile; a run's count is
// the difference of two numbers, each run adds (own << 32) | others to community c's cursor
// with one atomic, which hands it consecutive places in the segment, and a second walk over
// the entries writes them there.  Weighted: own-label weights are summed exactly per run and
// added to IWacc[c].
//
// STAGE_ROWS (a partition that does not follow the stored order, so that runs are hardly
// longer than a row): every row is a run, and every entry goes to its row's place, start +
// chunk prefix + per-node offset + its number in the row.
//
// Measured at 10M nodes and 200M entries: 242 us for a partition along the stored order, 338 for
// one that is not (584 and 1,171 when far labels were read at random from one XCD's L2, and
// every label from the row-major copy); 40M nodes, 400M entries: 934 us (2,736).
// What bounds it is a tile's chain of loads and barriers, hidden by one other workgroup per CU
// (32 waves, 64 registers each), and its instructions (one of a wave takes a SIMD 4 cycles): a
// bit more than 100M vector instructions at 10M nodes, 185 of the 242 us.  So the work per 64
// consecutive entries is kept to a few: a lane takes their places from 16-byte loads, one bit
// per entry says where a run starts, and an entry's run and its number among the staged ones
// are counts of bits below its lane.  What a wave needs for each of its (up to 24) vectors is
// held in its lanes and read as scalars.
enum { TG_BY_MODE = 0, TG_BY_ROWS = 1, TG_RUNS_ONLY = 2 };
template <class LT, bool WT>
struct TileLds {
  static constexpr int PER = 16 / (int)sizeof(LT);
  static constexpr int ARR = TG_ROWS + 8;
  static constexpr int VEC = TG_ENT / 64;
  // label table (window, up to fmax far labels); run starts and staged entries (a bit per
  // entry); per run place, label and first entry; run and number of every vector's first entry
  static constexpr int table(int fmax) { return (TG_WIN + fmax + PER - 1) / PER * 4; }
  static constexpr int words(int fmax) {
    return table(fmax) + 4 * VEC + ARR + ARR * (int)sizeof(LT) / 4 + ARR / 2 + VEC + (WT ? 4 * TG_ROWS : 0);
  }
  static constexpr size_t bytes(int fmax) { return 4 * (size_t)words(fmax); }
};

template <class LT, bool WT>
__global__ __launch_bounds__(TG_THREADS, 8) void k_tile_gather(
    int n, int t0, int T, int fmax, const Tile* __restrict__ tiles, const int32_t* __restrict__ rp, const uint16_t* __restrict__ eidx,
    const u32* __restrict__ fadr, const LT* __restrict__ fl, const LT* __restrict__ labx, const u32* __restrict__ start,
    const u32* __restrict__ D, unsigned long long* __restrict__ cur64, Ctl* __restrict__ ctl, LT* __restrict__ CB,
    const float* __restrict__ w, float* __restrict__ CW, unsigned long long* __restrict__ IWacc, int L, int chunk,
    const u32* __restrict__ PM, const u32* __restrict__ loc, int rows) {
  using TL = TileLds<LT, WT>;
  constexpr u32 NOLAB = (u32)LabelT<LT>::SENTINEL;
  constexpr u32 NOWHERE = 0x80000000u;  // places are below 2^31, and less an entry's number above -TG_ENT
  extern __shared__ __align__(16) u32 s_mem[];
  LT* s_tab = reinterpret_cast<LT*>(s_mem);
  u32* s_bits = s_mem + TL::table(fmax);  // 64 per vector: bit i - 1 for a run that starts at its entry i > 0
  unsigned long long* s_neq = reinterpret_cast<unsigned long long*>(s_bits + 2 * TL::VEC);
  u32* s_to = s_bits + 4 * TL::VEC;
  LT* s_lab = reinterpret_cast<LT*>(s_to + TL::ARR);
  uint16_t* s_first = reinterpret_cast<uint16_t*>(s_lab + TL::ARR);
  uint16_t* s_vrun = s_first + TL::ARR;
  uint16_t* s_vpre = s_vrun + TL::VEC;
  unsigned long long* s_ilo = reinterpret_cast<unsigned long long*>(s_vpre + TL::VEC);  // WT: own-label weight sum
  unsigned long long* s_ihi = s_ilo + TG_ROWS;
  __shared__ u32 s_last[TG_WAVES], s_heads[TG_WAVES], s_staged[TG_WAVES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto of = [](u32 x, int i) { return (u32)__builtin_amdgcn_readlane((int)x, i); };
  auto below_in = [](u32 lo, u32 hi, u32 base) {  // base + set bits below the lane
    return (u32)__builtin_amdgcn_mbcnt_hi((int)hi, __builtin_amdgcn_mbcnt_lo((int)lo, (int)base));
  };
  // each XCD (workgroup b runs on XCD b % 8) takes a contiguous eighth of the tiles
  const int per = (T + 7) / 8, t = (int)(blockIdx.x % 8u) * per + (int)(blockIdx.x / 8u);
  if ((int)(blockIdx.x / 8u) >= per || t >= T) return;
  const bool by_rows = !WT && sizeof(LT) == 2 && (rows == TG_BY_ROWS || ctl->mode == STAGE_ROWS);  // see k_colscan_rows
  if (by_rows && rows == TG_RUNS_ONLY) return;
  const Tile tile = tiles[t0 + t];
  const u32 ne = tile.ne;
  if (ne == 0) return;
  const int nrows = tile.r1 - tile.r0;
  const int w0 = tile_w0(tile.b0), w1 = tile_w1(tile.b0, n);
  // a wave takes `steps` consecutive groups
  const u32 ng = (ne + TG_GROUP - 1u) / TG_GROUP, steps = (ng + TG_WAVES - 1u) / TG_WAVES, gw = (u32)wv * steps;
  // every load that depends on no other first
  const int my_row = tile.r0 + min(tid, nrows - 1);
  const uint4* ew = reinterpret_cast<const uint4*>(eidx) + (size_t)tile.g0 * (TG_GROUP / 8);
  const u32* fp = fadr + tile.f0;
  constexpr int FU = 8;
  u32 fa[FU];
#pragma unroll
  for (int k = 0; k < FU; ++k) fa[k] = (u32)(tid + k * TG_THREADS) < tile.nf ? fp[(u32)(tid + k * TG_THREADS)] : 0u;
  uint4 q[TG_STEPS];
#pragma unroll
  for (int i = 0; i < TG_STEPS; ++i)
    q[i] = (u32)i < steps && gw + i < ng ? ew[(gw + i) * (u32)(TG_GROUP / 8) + lane] : make_uint4(0u, 0u, 0u, 0u);
  const u32 own = (u32)labx[(u32)my_row];
  const u32 ra = (u32)rp[(u32)my_row], rb = (u32)rp[(u32)my_row + 1u];
  const u32 lu = by_rows ? loc[(u32)my_row] : 0u;
  typedef u32 v4u __attribute__((ext_vector_type(4)));
  {
    const v4u* src = reinterpret_cast<const v4u*>(labx + w0);  // w0 is a multiple of 512; the array is padded past n
    v4u* dst = reinterpret_cast<v4u*>(s_mem);
    const u32 words = (u32)(w1 - w0 + TL::PER - 1) / TL::PER;
    for (u32 i = tid; i < words; i += TG_THREADS) dst[i] = src[i];
  }
  if (tid < 2 * TL::VEC) s_bits[tid] = 0;
  // the row's entries in the tile: [a, b)
  const u32 a = max(ra, tile.e0) - tile.e0, b = min(max(rb, tile.e0) - tile.e0, ne);
  const bool has = tid < nrows && a < b;
  const u64 hasm = __ballot(has);
  // the label of the wave's last row with entries
  if (hasm ? lane == 63 - __clzll((long long)hasm) : lane == 0) s_last[wv] = hasm ? own : SENT;
  {
    LT x[FU];
#pragma unroll
    for (int k = 0; k < FU; ++k)
      if ((u32)(tid + k * TG_THREADS) < tile.nf) x[k] = fl[fa[k]];
#pragma unroll
    for (int k = 0; k < FU; ++k)
      if ((u32)(tid + k * TG_THREADS) < tile.nf) s_tab[TG_WIN + tid + k * TG_THREADS] = x[k];
    for (u32 j = tid + FU * TG_THREADS; j < tile.nf; j += TG_THREADS) s_tab[TG_WIN + j] = fl[fp[j]];
  }
  // STAGE_ROWS: the place of the row's entry e, less e
  u32 row_to = NOWHERE;  // only with a label error, which voids the result
  if (by_rows && own != NOLAB && lu != SENT)
    row_to = start[own] + PM[(size_t)(my_row / chunk) * L + own] + lu + (tile.e0 - ra);
  __syncthreads();
  // runs
  u32 prev = SENT;
  {
    const u64 pm = hasm & ((1ull << lane) - 1ull);
    const u32 in_wave = (u32)__shfl((int)own, pm ? 63 - __clzll((long long)pm) : 0, 64);
    const u32 last = s_last[lane & (TG_WAVES - 1)];
    const u64 lm = __ballot(last != SENT) & ((1ull << wv) - 1ull);
    if (lm) prev = of(last, 63 - __clzll((long long)lm));
    if (pm) prev = in_wave;
  }
  const bool head = has && (by_rows || own != prev || prev == SENT);
  const u64 headm = __ballot(head);
  if (lane == 0) s_heads[wv] = (u32)__popcll(headm);
  __syncthreads();
  const u32 hincl = wave_incl_scan(lane < TG_WAVES ? s_heads[lane] : 0u);
  const u32 nruns = of(hincl, TG_WAVES - 1);
  // the row's run: heads up to and with the row, less 1
  const u32 run = below_in((u32)headm, (u32)(headm >> 32), (wv ? of(hincl, wv - 1) : 0u) + (head ? 1u : 0u)) - 1u;
  if (head) {
    s_first[run] = (uint16_t)a;
    s_lab[run] = (LT)own;
    if (by_rows) s_to[run] = row_to;
    if (a & 63u) atomicOr(&s_bits[2u * (a >> 6) + (((a & 63u) - 1u) >> 5)], 1u << (((a & 63u) - 1u) & 31u));
  }
  if (tid == 0) s_first[nruns] = (uint16_t)ne;
  if (has)
    for (u32 v = (a + 63u) / 64u; v * 64u < b; ++v) s_vrun[v] = (uint16_t)run;
  if (WT && tid < nrows) {
    s_ilo[tid] = 0ull;
    s_ihi[tid] = 0ull;
  }
  __syncthreads();
  // lane l: the wave's vector l
  const u32 v0 = gw * (TG_GROUP / 64);
  const bool have = (u32)lane < steps * (TG_GROUP / 64) && (v0 + lane) * 64u < ne;
  const u32 vl = v0 + (have ? (u32)lane : 0u);
  const u32 vbl = have ? s_bits[2u * vl] : 0u, vbh = have ? s_bits[2u * vl + 1u] : 0u, vr = have ? s_vrun[vl] : 0u;
  const u64 multi = __ballot((vbl | vbh) != 0u);
  auto half = [](const uint4& v, int k) {
    const u32 x = k < 2 ? v.x : k < 4 ? v.y : k < 6 ? v.z : v.w;
    return (k & 1) ? x >> 16 : x & 0xFFFFu;
  };
  auto label = [&](const uint4& v, int k) {
    return (u32) * reinterpret_cast<const LT*>(reinterpret_cast<const char*>(s_mem) + half(v, k) * (sizeof(LT) / 2));
  };
  if (by_rows) {
#pragma unroll
    for (int i = 0; i < TG_STEPS; ++i) {
      if ((u32)i >= steps || gw + i >= ng) break;
      u32 to[8], x[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int v = 8 * i + k;
        to[k] = s_to[below_in(of(vbl, v), of(vbh, v), of(vr, v))];
        x[k] = label(q[i], k);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const u32 e = (gw + i) * TG_GROUP + (u32)(64 * k + lane);
        if (to[k] != NOWHERE && e < ne) CB[to[k] + e] = (LT)x[k];
      }
    }
    return;
  }
  // what the claims need of their communities
  const u32 c = (u32)tid < nruns ? (u32)s_lab[tid] : NOLAB;
  const u32 dc = c != NOLAB ? D[c] : 0u, sc = c != NOLAB ? start[c] : 0u;
  // first walk: which entries are staged
  const u32 vc = have ? (u32)s_lab[vr] : 0u;
  u32 nlo = 0, nhi = 0;  // lane l: the staged entries of vector l
#pragma unroll
  for (int i = 0; i < TG_STEPS; ++i) {
    if ((u32)i >= steps || gw + i >= ng) break;
    const u32 e0 = (gw + i) * TG_GROUP;
    u32 x[8];
    u64 m[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = label(q[i], k);
    if ((multi >> (8 * i)) & 0xFFull) {
      u32 c[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) c[k] = (u32)s_lab[below_in(of(vbl, 8 * i + k), of(vbh, 8 * i + k), of(vr, 8 * i + k))];
#pragma unroll
      for (int k = 0; k < 8; ++k) m[k] = __ballot(x[k] != c[k]);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) m[k] = __ballot(x[k] != of(vc, 8 * i + k));
    }
    if (ne - e0 < (u32)TG_GROUP) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const u32 left = ne - e0 > 64u * k ? ne - e0 - 64u * k : 0u;
        if (left < 64u) m[k] &= (1ull << left) - 1ull;
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const bool it = __builtin_amdgcn_inverse_ballot_w64(1ull << (8 * i + k));
      nlo = it ? (u32)m[k] : nlo;
      nhi = it ? (u32)(m[k] >> 32) : nhi;
    }
    if (sizeof(LT) == 2)  // the labels take the places' registers
      q[i] = make_uint4(x[0] | x[1] << 16, x[2] | x[3] << 16, x[4] | x[5] << 16, x[6] | x[7] << 16);
  }
  u32 vp;
  {
    const u32 cnt = (u32)(__popc(nlo) + __popc(nhi)), incl = wave_incl_scan(cnt);
    vp = incl - cnt;
    if (have) {
      s_neq[vl] = ((u64)nhi << 32) | nlo;
      s_vpre[vl] = (uint16_t)vp;
    }
    if (lane == 63) s_staged[wv] = incl;
  }
  __syncthreads();
  // number of the first staged entry of every wave
  const u32 wincl = wave_incl_scan(lane < TG_WAVES ? s_staged[lane] : 0u);
  vp += wv ? of(wincl, wv - 1) : 0u;
  // one claim per run
  {
    // staged entries before entry e of the tile
    const bool mine = (u32)tid < nruns;
    auto before = [&](u32 e) {
      const u32 v = min(e, ne - 1u) >> 6, wave = v / (steps * (TG_GROUP / 64));
      const u32 base = (u32)__shfl((int)wincl, wave ? (int)wave - 1 : 0, 64);
      return (wave ? base : 0u) + s_vpre[v] +
             (e >= ne ? (u32)__popcll(s_neq[v]) : (u32)__popcll(s_neq[v] & ((1ull << (e & 63u)) - 1ull)));
    };
    const u32 f = mine ? (u32)s_first[tid] : 0u, z = mine ? (u32)s_first[tid + 1] : 0u;
    const u32 p = before(f), inter = before(z) - p;
    if (mine) {
      const u32 tot = z - f;
      u32 to = NOWHERE;
      if (c != NOLAB) {
        const unsigned long long old = atomicAdd(&cur64[c], ((unsigned long long)(tot - inter) << 32) | inter);
        const u32 lo = (u32)old;
        if (lo + inter <= dc) to = sc + lo - p;
        else atomicOr(&ctl->flags, F_SEGMENT);  // never expected: the tile's counts disagree with the degrees
      }
      s_to[tid] = to;
    }
  }
  __syncthreads();
  // second walk: their labels (and weights) to their places
  const u32 vt = have ? s_to[vr] : NOWHERE;
#pragma unroll
  for (int i = 0; i < TG_STEPS; ++i) {
    if ((u32)i >= steps || gw + i >= ng) break;
    const u32 e0 = (gw + i) * TG_GROUP;
    u32 to[8];
    if ((multi >> (8 * i)) & 0xFFull) {
#pragma unroll
      for (int k = 0; k < 8; ++k) to[k] = s_to[below_in(of(vbl, 8 * i + k), of(vbh, 8 * i + k), of(vr, 8 * i + k))];
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k) to[k] = of(vt, 8 * i + k);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const u32 lo = of(nlo, 8 * i + k), hi = of(nhi, 8 * i + k);
      const u32 at = below_in(lo, hi, to[k] + of(vp, 8 * i + k));
      if (__builtin_amdgcn_inverse_ballot_w64(((u64)hi << 32) | lo) && to[k] != NOWHERE) {
        CB[at] = (LT)(sizeof(LT) == 2 ? half(q[i], k) : label(q[i], k));
      }
    }
  }
  if constexpr (WT) {
    // every weight once: a staged entry's to its place, an own-label entry's into its run's sum.
    // A vector inside one run adds in registers, reduced once per run; in a vector of several runs
    // every lane adds to its run's words in LDS (a reduction per run took most of the pass where
    // runs are short: 2M nodes, 40M entries and labels that change every few rows 195 us, now 164).
    u32 wrun = SENT;  // the run whose own-label weights wacc sums
    WeightSum wacc;
    auto add_to_run = [&](u32 r, u64 lo, u64 hi) {
      const u64 old = atomicAdd(&s_ilo[r], lo);
      hi += old + lo < old ? 1ull : 0ull;
      if (hi) atomicAdd(&s_ihi[r], hi);
    };
    auto wflush = [&]() {
      if (wrun == SENT) return;
      const u128 sum = wave_sum_u128(wacc.value());
      if (lane == 0) add_to_run(wrun, (u64)sum, (u64)(sum >> 64));
      wacc = WeightSum();
    };
    constexpr int U = 8;  // loads in flight
    const int nv = (int)min(steps * (u32)(TG_GROUP / 64), v0 * 64u < ne ? (ne - v0 * 64u + 63u) / 64u : 0u);
    for (int vb = 0; vb < nv; vb += U) {
      float wt[U];
#pragma unroll
      for (int k = 0; k < U; ++k) wt[k] = w[tile.e0 + min((v0 + (u32)(vb + k)) * 64u + (u32)lane, ne - 1u)];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int v = vb + k;
        if (v >= nv) break;
        const u32 slo = of(nlo, v), shi = of(nhi, v), bl = of(vbl, v), bh = of(vbh, v);
        const bool several = (bl | bh) != 0u;  // uniform
        const u32 r = several ? below_in(bl, bh, of(vr, v)) : of(vr, v);
        const u32 to = several ? s_to[r] : of(vt, v);
        const bool staged = __builtin_amdgcn_inverse_ballot_w64(((u64)shi << 32) | slo);
        if (staged && to != NOWHERE) CW[below_in(slo, shi, to + of(vp, v))] = wt[k];
        const bool mine = !staged && (v0 + (u32)v) * 64u + (u32)lane < ne;
        u64 vlo, vhi;
        WeightSum::split(wt[k], vlo, vhi);
        if (several) {
          if (mine) add_to_run(r, vlo, vhi);
        } else if (__ballot(mine)) {
          if (r != wrun) {
            wflush();
            wrun = r;
          }
          if (mine) wacc.add(vlo, vhi);
        }
      }
    }
    wflush();
    __syncthreads();
    if (c != NOLAB) {  // a run's thread
      const unsigned long long ilo = s_ilo[tid], ihi = s_ihi[tid];
      if (ilo | ihi) {
        const unsigned long long was = atomicAdd(&IWacc[2 * (size_t)c], ilo);
        const unsigned long long h = ihi + (was + ilo < was ? 1ull : 0ull);
        if (h) atomicAdd(&IWacc[2 * (size_t)c + 1], h);
      }
    }
  }
}

}  // namespace cq
