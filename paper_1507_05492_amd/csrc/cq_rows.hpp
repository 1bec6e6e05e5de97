// Scoring a partition by member rows (Section II-B): for graphs whose staged labels fit one
// XCD's L2 the neighbour labels are not staged into community segments at all.  The nodes
// are sorted by community (a counting sort: one record (first entry, degree) per node), and
// the group pass walks the rows of a community's members itself, reads each neighbour's
// label and counts it in the community's LDS table.  Against the edge pass this leaves out
// the write and the second read of every staged label and the per-entry search over the
// rows of a tile; what remains is one label read per entry, which L2 serves at 265 G/s
// whatever the order of the nodes (measured: random 2-byte reads over 1 to 4 MB; 77 G/s over
// 20 MB and 58 G/s over 80 MB, where the coalesced edge passes are the better choice).
#pragma once

namespace cq {

// Counting sort, pass 1: labels in the stored order (labx), each node's rank among its
// chunk's nodes of the same label (loc), and the chunk's nodes per label (row blockIdx.x of
// HN).  A label out of range is staged as the sentinel and reported in bad[blockIdx.x].
// Workgroup 0 also clears the control block and sets every work queue's ticket counter to
// first_tickets (the group pass's workgroups take their first community without a ticket).
constexpr int RN_UNROLL = 4;
template <class LT>
__global__ __launch_bounds__(1024) void k_rows_node(int n, const int32_t* __restrict__ labels, const int32_t* __restrict__ perm,
                                                    int L, int chunk, u32* __restrict__ HN, u32* __restrict__ loc,
                                                    LT* __restrict__ labx, u32* __restrict__ bad, Ctl* __restrict__ ctl,
                                                    u32* __restrict__ wq, u32 first_tickets) {
  extern __shared__ u32 s_hist[];
  __shared__ u32 s_bad;
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    for (u32 i = tid; i < sizeof(Ctl) / 4; i += 1024) reinterpret_cast<u32*>(ctl)[i] = 0;
    for (u32 i = tid; i < WQ_WORDS; i += 1024) wq[i] = i < WQ_QUEUES * WQ_LINE && i % WQ_LINE == 0 ? first_tickets : 0u;
  }
  for (int i = tid; i < L; i += 1024) s_hist[i] = 0;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  const long long u0 = (long long)blockIdx.x * chunk;
  const long long u1 = min((long long)n, u0 + chunk);
  u32 wrong = 0;
  for (long long ub = u0; ub < u1; ub += 1024 * RN_UNROLL) {  // uniform trip count
    long long u[RN_UNROLL];
    int c[RN_UNROLL];
#pragma unroll
    for (int k = 0; k < RN_UNROLL; ++k) {
      u[k] = ub + tid + (long long)k * 1024;
      c[k] = u[k] < u1 ? (perm ? perm[u[k]] : (int)u[k]) : -1;
    }
#pragma unroll
    for (int k = 0; k < RN_UNROLL; ++k)
      if (u[k] < u1) c[k] = labels[c[k]];
#pragma unroll
    for (int k = 0; k < RN_UNROLL; ++k) {
      const bool in = u[k] < u1;
      const bool ok = in && (u32)c[k] < (u32)L;
      wrong |= in && !ok;
      const u32 rank = wave_count<4>(s_hist, (u32)c[k], ok);
      if (in) {
        loc[u[k]] = rank;
        labx[u[k]] = ok ? (LT)c[k] : LabelT<LT>::SENTINEL;
      }
    }
  }
  if (wrong) s_bad = 1;
  __syncthreads();
  for (int c = tid; c < L; c += 1024) HN[(size_t)blockIdx.x * L + c] = s_hist[c];
  if (tid == 0) bad[blockIdx.x] = s_bad;
}

// A community of at least 2^split nodes is shared by several workgroups of the group pass, a
// part of `part` members each.  Their counts meet in a row of the split table: the counters per
// label, then own-label entries, degree sum and finished parts.
__host__ __device__ constexpr u32 rg_row_words(u32 L) { return ((L + 3u) & ~3u) + 4u; }

// Pass 2: chunk prefixes (in HN) and totals N per label; the last workgroup to finish builds
// the segment starts, the work order (by decreasing node count) and the list of parts (index
// of the community in the order << 16 | part), and sets the flags.
__global__ __launch_bounds__(CS_LABELS * CS_GROUPS) void k_rows_scan(int W, int L, u32* __restrict__ HN, u32* __restrict__ N,
                                                                     u32* __restrict__ start, u32* __restrict__ order,
                                                                     u32* __restrict__ parts, int split, u32 part,
                                                                     const u32* __restrict__ bad, Ctl* __restrict__ ctl) {
  static_assert(CS_LABELS * CS_GROUPS == 1024, "scan_order_body");
  __shared__ u32 s_w[SCAN_THREADS / 64];
  colscan_tile<false, true>(W, L, HN, HN, N, nullptr, nullptr, blockIdx.x);
  if (!last_workgroup(&ctl->done, gridDim.x)) return;
  const u32 kbig = scan_order_body(L, N, N, start, order, ctl, split + 1);  // at most n >> split, fewer than 1,024
  u32 wrong = 0;
  for (int w = threadIdx.x; w < W; w += 1024) wrong |= bad[w];
  if (wrong) ctl->flags = F_LABEL;
  if (kbig == 0) return;  // ctl->parts stays 0
  __syncthreads();        // the order is written
  const u32 mine = threadIdx.x < kbig ? (N[order[threadIdx.x]] + part - 1u) / part : 0u;
  u32 total;
  const u32 at = block_excl_scan_1024(mine, s_w, &total);
  for (u32 j = 0; j < mine; ++j) parts[at + j] = threadIdx.x << 16 | j;
  if (threadIdx.x == 0) ctl->parts = total;
}

// Pass 3: the members' records, community by community: (first entry, degree) of node u at
// start[c] + chunk prefix + rank.  Clears the split table's rows on the way.
template <class LT>
__global__ __launch_bounds__(256) void k_rows_place(int n, const int32_t* __restrict__ rp, int L, int chunk,
                                                    const u32* __restrict__ HN, const u32* __restrict__ start,
                                                    const u32* __restrict__ loc, const LT* __restrict__ labx,
                                                    uint2* __restrict__ rec, u32* __restrict__ table, const Ctl* __restrict__ ctl) {
  for (long long u = (long long)blockIdx.x * 256 + threadIdx.x; u < n; u += (long long)gridDim.x * 256) {
    const LT c = labx[u];
    if (c == LabelT<LT>::SENTINEL) continue;
    const u32 b = (u32)rp[u], e = (u32)rp[u + 1];
    rec[start[c] + HN[(size_t)(u / chunk) * L + c] + loc[u]] = make_uint2(b, e - b);
  }
  const u32 words = ctl->kbig * rg_row_words((u32)L);
  for (u32 i = blockIdx.x * 256u + threadIdx.x; i < words; i += gridDim.x * 256u) table[i] = 0;
}

// Group pass over member rows.  A workgroup of NT threads takes a community (or a part of a
// large one); each of its waves takes up to 64 members at a time, scans their degrees, and
// walks their entries 64 at a time, RG_UNROLL steps in flight: an entry's row is found by a
// six-step search over the wave's 64 row starts in LDS.  Rows of RG_HUB entries and more are
// left for all waves to walk together afterwards (2M nodes, a hub joined to all of them: 9.9 ms
// a call when one wave walked its row, 0.46 by the workgroup; staged 9.2).  The counts go to a direct LDS table (L <=
// lds_words); the table is visited by the first NTV threads in the same fixed order as in
// group_one, so the results do not depend on NT, nor on the pass that counted.  The parts of
// a large community add their tables in its row of the split table, and the last one visits
// the sums.  D[g] (the degree sum) is written here as well.  Items (parts first, then the
// other communities in order) come from the work queues; a workgroup's first one is its own
// number.
constexpr int RG_UNROLL = 8;
constexpr u32 RG_HUB = 4096;
constexpr u32 RG_HUBS = 64;  // hubs of one item; further ones are walked by their wave
template <class LT, int NT, int NTV>
__global__ __launch_bounds__(NT, 8) void k_rows_groups(const uint2* __restrict__ rec, const int32_t* __restrict__ col,
                                                    const LT* __restrict__ labx, const u32* __restrict__ start,
                                                    const u32* __restrict__ order, u32* __restrict__ D,
                                                    Ctl* __restrict__ ctl, u32 Lv, ScoreVis vis, u32* __restrict__ wq,
                                                    const u32* __restrict__ parts, u32 part, u32* __restrict__ table) {
  static_assert(NTV <= NT, "the visiting threads are the first of the workgroup");
  extern __shared__ __align__(16) u32 tab[];
  __shared__ u32 s_ex[NT], s_off[NT];  // per wave: row starts among its 64 rows' entries, and column index minus that
  __shared__ uint2 s_hub[RG_HUBS];
  __shared__ u32 s_hot, s_deg, s_item, s_hubs;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  u32* ex = s_ex + wv * 64;
  u32* off = s_off + wv * 64;
  const u32 P = ctl->parts, kbig = ctl->kbig;
  const u32 K = P + (ctl->K - kbig);
  u32 item = blockIdx.x;
  u32 q = blockIdx.x % WQ_QUEUES, left = WQ_QUEUES;  // thread 0's queue state (see wq_next)
  const u32 nq = (Lv + 3u) >> 2;
  uint4* tab4 = reinterpret_cast<uint4*>(tab);
  while (item < K) {  // uniform
    u32 code = 0;  // of a part
    if (item < P) code = parts[item];
    const u32 g = order[item < P ? code >> 16 : item - P + kbig];
    const u32 ng = vis.N[g];
    u32 m0 = start[g], nm = ng;
    if (item < P) {
      const u32 first = (code & 0xFFFFu) * part;
      m0 += first;
      nm = min(part, ng - first);
    }
    for (u32 i = tid; i < nq; i += NT) tab4[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) {
      s_hot = 0;
      s_deg = 0;
      s_hubs = 0;
    }
    __syncthreads();
    // members per wave and step: all waves share a small community
    u32 mc = (nm + NT / 64 - 1) / (NT / 64);
    mc = min(64u, max(4u, mc));
    u32 mine = 0, deg = 0;
    // counts the entries at[k] with e + step * k < end; all loads are issued before the first use
    auto count = [&](const u32 (&at)[RG_UNROLL], u32 e, u32 step, u32 end) {
      u32 v[RG_UNROLL], x[RG_UNROLL];
#pragma unroll
      for (int k = 0; k < RG_UNROLL; ++k) v[k] = (u32)col[at[k]];
#pragma unroll
      for (int k = 0; k < RG_UNROLL; ++k) x[k] = (u32)labx[v[k]];
#pragma unroll
      for (int k = 0; k < RG_UNROLL; ++k) {
        if (e + step * (u32)k < end) {
          if (x[k] == g) ++mine;
          else if (x[k] < Lv) atomicAdd(&tab[x[k]], 1u);
        }
      }
    };
    for (u32 m = wv * mc; m < nm; m += (NT / 64) * mc) {
      const bool has = (u32)lane < mc && m + lane < nm;
      uint2 r = make_uint2(0u, 0u);
      if (has) r = rec[m0 + m + lane];
      if (r.y >= RG_HUB) {
        const u32 h = atomicAdd(&s_hubs, 1u);
        if (h < RG_HUBS) {
          s_hub[h] = r;
          atomicAdd(&s_deg, r.y);
          r.y = 0;
        }
      }
      const u32 incl = wave_incl_scan(r.y);
      const u32 tot = __shfl(incl, 63, 64);
      deg += tot;
      ex[lane] = incl - r.y;  // lanes without a row: tot, which no entry reaches
      off[lane] = r.x - (incl - r.y);
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      for (u32 eb = lane; eb < tot; eb += 64 * RG_UNROLL) {
        u32 at[RG_UNROLL];
#pragma unroll
        for (int k = 0; k < RG_UNROLL; ++k) {
          const u32 e = min(eb + 64u * (u32)k, tot - 1u);  // in bounds; masked below
          u32 l = 0;  // last row with ex[l] <= e
#pragma unroll
          for (u32 s = 32; s > 0; s >>= 1)
            if (ex[l + s] <= e) l += s;
          at[k] = e + off[l];
        }
        count(at, eb, 64u, tot);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    mine = wave_sum_u32(mine);
    if (lane == 0) {
      if (mine) atomicAdd(&s_hot, mine);
      if (deg) atomicAdd(&s_deg, deg);
    }
    // the next item's ticket is taken before the visits
    if (tid == 0) s_item = gridDim.x >= K ? K : wq_next(wq, K, q, left);
    __syncthreads();
    if (const u32 hubs = min(s_hubs, RG_HUBS)) {  // uniform
      mine = 0;
      for (u32 h = 0; h < hubs; ++h) {
        const uint2 r = s_hub[h];
        for (u32 eb = tid; eb < r.y; eb += NT * RG_UNROLL) {
          u32 at[RG_UNROLL];
#pragma unroll
          for (int k = 0; k < RG_UNROLL; ++k) at[k] = r.x + min(eb + (u32)NT * (u32)k, r.y - 1u);
          count(at, eb, (u32)NT, r.y);
        }
      }
      mine = wave_sum_u32(mine);
      if (lane == 0 && mine) atomicAdd(&s_hot, mine);
      __syncthreads();
    }
    const u32 next = s_item;
    bool visits = true;
    if (item < P) {
      u32* row = table + (size_t)(code >> 16) * rg_row_words(Lv);
      u32* sums = row + rg_row_words(Lv) - 4u;
      u32 t = tid;
      asm volatile("" : "+v"(t));  // addresses from it are formed here, not kept in registers through the item loop
      for (u32 i = t; i < Lv; i += NT)
        if (tab[i]) atomicAdd(&row[i], tab[i]);
      if (tid == 0) {
        atomicAdd(&sums[0], s_hot);
        atomicAdd(&sums[1], s_deg);
      }
      visits = last_workgroup(&sums[2], (ng + part - 1u) / part);
      if (visits) {
        for (u32 i = t; i < nq; i += NT) tab4[i] = reinterpret_cast<const uint4*>(row)[i];
        if (tid == 0) {
          s_hot = sums[0];
          s_deg = sums[1];
        }
        __syncthreads();
      }
    }
    if (visits) {
      ScoreVis::State st;
      vis.begin_n(st, g, ng);
      if (tid == 0) {
        D[g] = s_deg;
        if (s_hot) vis.visit(st, g, s_hot);
      }
      if (tid < NTV) visit_direct<NTV>(tab4, nq, st, vis);
      vis.settle(st);
      vis.finish(st, g);
    }
    __syncthreads();
    item = next;
  }
}

}  // namespace cq
