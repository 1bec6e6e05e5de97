// cq_device.hpp -- device-side building blocks shared by the gfx950 kernels:
// integer types, exact fixed-point accumulation, wave/block reductions and the
// per-workgroup LDS count tables (direct-indexed and open-addressing).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cq {

typedef unsigned __int128 u128;
typedef uint64_t u64;
typedef uint32_t u32;

constexpr u32 SENT = 0xFFFFFFFFu;  // "no label" marker in staged label arrays
constexpr u32 EMPTY = 0xFFFFFFFFu; // empty hash slot

// device flag bits (cq_score_result.device_flags / cq_compare_result.device_flags)
constexpr u32 F_LABEL = 1u;   // a label outside [0, num_labels)
constexpr u32 F_GRAPH = 2u;   // malformed CSR (graph load only)
constexpr u32 F_EXPORT = 4u;  // export table too small
constexpr u32 F_STACK = 8u;   // internal: class stack exhausted (never expected)
constexpr u32 F_SEGMENT = 16u;  // internal: a community's entries exceed its segment (never expected)

// Control block at the start of every workspace.
struct Ctl {
  u32 flags;
  u32 K;          // non-empty communities (filled by the scan kernel)
  u32 kbig;       // groups whose segment holds at least GW_SPLIT entries (they come first in the order)
  u32 dense_rows;  // node pass of tiled graphs: buckets that wrote histogram rows
  unsigned long long export_count;
  u32 done, done2;  // workgroups that have finished a pass whose last workgroup goes on alone
  u32 changes;    // tiled graphs' node pass: label changes between consecutive stored ids
  u32 mode;       // tiled graphs: STAGE_BLOCKS or STAGE_ROWS, chosen from `changes`
  u32 parts;      // member rows: parts of the kbig communities that several workgroups share;
                  // comparison by bins: slices of the large bins
  u32 pad0;
  unsigned long long pad1[2];
};

// ---- work queues of the persistent per-community kernels ----------------------
// Atomics on one address are serialised where they are performed (about 12 ns each,
// measured on MI355X), so a single ticket counter caps a persistent kernel at one item
// per 12 ns however many workgroups wait.  The K items of an ordered list are therefore
// split into WQ_QUEUES interleaved queues (queue q hands out items q, q + 8, q + 16, ...,
// so each keeps the list's order), each with its counter on its own 128-byte line.  A
// workgroup starts on queue blockIdx.x % 8 (workgroups are dealt to the XCDs in turn)
// and moves on to the next queue when its own is empty, so none exits while work is left.
constexpr u32 WQ_QUEUES = 8;
constexpr u32 WQ_LINE = 32;                    // u32 words per counter line (128 bytes)
// tickets of the workgroup-per-group pass, per-queue 64-bit sums (cells), tickets of the
// wave-per-group pass
constexpr u32 WQ_WORDS = 3 * WQ_QUEUES * WQ_LINE;
constexpr size_t WQ_BYTES = 4 * (size_t)WQ_WORDS;
constexpr u32 WQ_WAVE = 2 * WQ_QUEUES * WQ_LINE;  // word offset of the wave pass's tickets

// Next item for the calling workgroup (thread 0 only), or 0xFFFFFFFF when every queue is
// empty.  q and left are thread 0's own state: start with q = blockIdx.x % 8, left = 8.
__device__ __forceinline__ u32 wq_next(u32* __restrict__ wq, u32 K, u32& q, u32& left) {
  while (left) {
    const u32 i = atomicAdd(&wq[q * WQ_LINE], 1u);
    const u64 item = (u64)q + (u64)WQ_QUEUES * i;
    if (item < K) return (u32)item;
    q = (q + 1u) % WQ_QUEUES;
    --left;
  }
  return 0xFFFFFFFFu;
}
// a 64-bit sum kept per queue on its own line (the second half of the region)
__device__ __forceinline__ unsigned long long* wq_sum(u32* wq, u32 q) {
  return reinterpret_cast<unsigned long long*>(wq + (WQ_QUEUES + q) * WQ_LINE);
}

// How a call on a tiled graph stages the neighbour labels (Ctl::mode; also reported in the
// result): with run claims, or at per-node offsets when the partition does not follow the
// stored order (short runs of equal labels make run claims as many as the nodes).
constexpr u32 STAGE_ROWS_ONLY = 0;  // the graph has no tiles
constexpr u32 STAGE_BLOCKS = 1;
constexpr u32 STAGE_ROWS = 2;

// ---- exact fixed-point accumulation --------------------------------------
// A binary64 value t is turned into the integer round_toward_zero(t * 2^96) held in
// a 128-bit two's-complement word.  Integer addition is associative, so sums of
// such words are independent of the order in which terms arrive.  |t| < 2^31 is
// required; every term accumulated this way is bounded far below that.
__device__ __forceinline__ u128 fix96(double t) {
  double a = fabs(t);
  double f = ldexp(a, 96);
  u64 hi = __double2ull_rz(ldexp(f, -64));
  double rem = f - ldexp((double)hi, 64);  // exact: f and hi*2^64 share the leading bits
  u64 lo = __double2ull_rz(rem);
  u128 v = ((u128)hi << 64) | (u128)lo;
  return t < 0 ? (u128)(-(__int128)v) : v;
}
__device__ __forceinline__ double unfix96(u128 v) {
  bool neg = ((__int128)v) < 0;
  u128 a = neg ? (u128)(-(__int128)v) : v;
  double d = ldexp((double)(u64)(a >> 64), -32) + ldexp((double)(u64)a, -96);
  return neg ? -d : d;
}

// The same truncation, floor(t * 2^96), for terms known to lie in [0, 1), accumulated as
// three 32-bit limbs of the fraction in 64-bit words (fewer instructions than fix96).
struct Frac96Sum {
  u64 a = 0, b = 0, c = 0;
  __device__ __forceinline__ void add(double t) {
    const double x = t * 4294967296.0;  // 2^32
    const u32 l0 = (u32)x;               // truncation; each remainder below is exact
    const double y = (x - (double)l0) * 4294967296.0;
    const u32 l1 = (u32)y;
    const double z = (y - (double)l1) * 4294967296.0;
    const u32 l2 = (u32)z;
    a += l0;
    b += l1;
    c += l2;
  }
  // t in [0, 2^20): the integer part joins the first limb as well
  __device__ __forceinline__ void add_wide(double t) {
    const double x = t * 4294967296.0;
    const u64 l0 = (u64)x;
    const double y = (x - (double)l0) * 4294967296.0;
    const u32 l1 = (u32)y;
    const double z = (y - (double)l1) * 4294967296.0;
    const u32 l2 = (u32)z;
    a += l0;
    b += l1;
    c += l2;
  }
  __device__ __forceinline__ u128 value() const { return ((u128)a << 64) + ((u128)b << 32) + (u128)c; }
};

// 1/y for finite y >= 1: the hardware reciprocal estimate refined by two Newton-Raphson
// steps (r <- r + r(1 - yr), each squaring the relative error), which leaves it within
// about one unit in the last place; unlike a division it need not be correctly rounded.
__device__ __forceinline__ double recip_nr(double y) {
  double r = __builtin_amdgcn_rcp(y);
  double e = __builtin_fma(-y, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-y, r, 1.0);
  return __builtin_fma(r, e, r);
}

// ---- exact edge-weight sums --------------------------------------------------
// A float32 weight w in [2^-32, 2^32] is its 24-bit significand times 2^(e - 150), e the
// biased exponent (95 <= e <= 159), so w * 2^55 is the integer significand << (e - 95),
// below 2^88.  Sums of such integers are exact and independent of order, and 2^31 of
// them stay below 2^119.
constexpr float WEIGHT_MIN = 2.3283064365386963e-10f;  // 2^-32
constexpr float WEIGHT_MAX = 4294967296.0f;            // 2^32
constexpr u32 WEIGHT_EXP0 = 95;                        // biased exponent of 2^-32
__device__ __forceinline__ u128 fixw_f32(float w) {
  const u32 b = __float_as_uint(w);
  const u32 e = (b >> 23) & 0xFFu;
  return (u128)((b & 0x7FFFFFu) | 0x800000u) << (e - WEIGHT_EXP0);
}
// Exact sum of float32 weights in [WEIGHT_MIN, WEIGHT_MAX], times 2^55 (the value of
// fixw_f32), in two 64-bit words.  split() gives a weight's fixed-point value as
// (hi, lo): its 24-bit significand shifted left by s = biased exponent - WEIGHT_EXP0
// (0 <= s <= 64).
struct WeightSum {
  u64 lo = 0, hi = 0;
  static __device__ __forceinline__ void split(float w, u64& vlo, u64& vhi) {
    const u32 b = __float_as_uint(w);
    const u32 sh = ((b >> 23) & 0xFFu) - WEIGHT_EXP0;
    const u64 sig = (u64)((b & 0x7FFFFFu) | 0x800000u);
    vlo = sh < 64u ? sig << sh : 0ull;
    vhi = sh > 40u ? sig >> (64u - sh) : 0ull;
  }
  __device__ __forceinline__ void add(u64 vlo, u64 vhi) {
    lo += vlo;
    hi += vhi + (lo < vlo ? 1ull : 0ull);
  }
  __device__ __forceinline__ u128 value() const { return ((u128)hi << 64) | lo; }
};

// value / 2^55 of an exact weight sum
__device__ __forceinline__ double unfixw(u128 v) {
  return (double)(u64)(v >> 64) * 512.0 + (double)(u64)v * 2.7755575615628914e-17;  // 2^9, 2^-55
}

// ---- wave / block reductions (wave64) ---------------------------------------
// Every lane of the wave must be active.  A sum of 64 lanes is a butterfly: lanes 32, 16, 8,
// 4, 2 and 1 apart exchange values.  The exchanges are lane swaps and DPP moves of a few
// cycles; as LDS permutes (__shfl_xor) each step waited for the LDS (about 100 cycles), and
// the reductions were most of the kernels that finish a small call.
template <int CTRL>
__device__ __forceinline__ u32 dpp_u32(u32 x) {
  return (u32)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
// the value of lane ^ M (M = 1, 2, 4, 8)
template <int M>
__device__ __forceinline__ u32 lane_xor(u32 x) {
  if constexpr (M == 1) return dpp_u32<0xB1>(x);        // quad_perm [1,0,3,2]
  else if constexpr (M == 2) return dpp_u32<0x4E>(x);   // quad_perm [2,3,0,1]
  else if constexpr (M == 4) return dpp_u32<0x1B>(dpp_u32<0x141>(x));  // row_half_mirror, then quad_perm [3,2,1,0]
  else return dpp_u32<0x128>(x);                        // row_ror:8
}
// the values of the lanes 32 (16) apart as an unordered pair, the same pair in both lanes
__device__ __forceinline__ void pair32(u32 x, u32& a, u32& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  a = r[0];
  b = r[1];
}
__device__ __forceinline__ void pair16(u32 x, u32& a, u32& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  a = r[0];
  b = r[1];
}
// Butterfly over T (words of 32 bits) with a commutative operation f(T, T).
template <class T, class F>
__device__ __forceinline__ T wave_butterfly(T x, F f) {
  constexpr int W = sizeof(T) / 4;
  struct Words { u32 w[W]; };
  auto step = [&](auto exchange) {
    const Words v = __builtin_bit_cast(Words, x);
    Words a, b;
#pragma unroll
    for (int i = 0; i < W; ++i) exchange(v.w[i], a.w[i], b.w[i]);
    x = f(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
  };
  step([](u32 v, u32& a, u32& b) { pair32(v, a, b); });
  step([](u32 v, u32& a, u32& b) { pair16(v, a, b); });
  step([](u32 v, u32& a, u32& b) { a = v; b = lane_xor<8>(v); });
  step([](u32 v, u32& a, u32& b) { a = v; b = lane_xor<4>(v); });
  step([](u32 v, u32& a, u32& b) { a = v; b = lane_xor<2>(v); });
  step([](u32 v, u32& a, u32& b) { a = v; b = lane_xor<1>(v); });
  return x;
}
__device__ __forceinline__ u64 wave_sum_u64(u64 x) {
  return wave_butterfly(x, [](u64 a, u64 b) { return a + b; });
}
__device__ __forceinline__ u32 wave_sum_u32(u32 x) {
  return wave_butterfly(x, [](u32 a, u32 b) { return a + b; });
}
__device__ __forceinline__ u64 wave_max_u64(u64 x) {
  return wave_butterfly(x, [](u64 a, u64 b) { return a > b ? a : b; });
}
__device__ __forceinline__ u32 wave_max_u32(u32 x) {
  return wave_butterfly(x, [](u32 a, u32 b) { return a > b ? a : b; });
}
__device__ __forceinline__ double wave_max_f64(double x) {
  return wave_butterfly(x, [](double a, double b) { return a > b ? a : b; });
}
__device__ __forceinline__ double wave_sum_f64(double x) {
  return wave_butterfly(x, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ u128 wave_sum_u128(u128 x) {
  struct P { u64 lo, hi; };
  const P r = wave_butterfly(P{(u64)x, (u64)(x >> 64)}, [](P a, P b) {
    const u64 lo = a.lo + b.lo;
    return P{lo, a.hi + b.hi + (lo < a.lo ? 1ull : 0ull)};
  });
  return ((u128)r.hi << 64) | r.lo;
}
// inclusive scan of u32 inside a wave (row shifts, then each row's last lane added to the rows after it)
__device__ __forceinline__ u32 wave_incl_scan(u32 x) {
  x += dpp_u32<0x111>(x);  // row_shr:1
  x += dpp_u32<0x112>(x);
  x += dpp_u32<0x114>(x);
  x += dpp_u32<0x118>(x);
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15 to rows 1 and 3
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31 to rows 2 and 3
  return x;
}

// Adds one to the LDS counter s[bin] for every lane with `on`; returns the counter's value
// before this lane's own addition.  Atomics on one LDS address are performed one after
// another, so up to ROUNDS times the lanes that share the first pending lane's bin (nodes
// stored by community), when there are at least four of them, add through one lane.  The
// calling wave must be converged.
template <int ROUNDS>
__device__ __forceinline__ u32 wave_count(u32* s, u32 bin, bool on) {
  const u32 lane = threadIdx.x & 63u;
  u32 old = 0;
  for (int i = 0; i < ROUNDS; ++i) {
    const u64 act = __ballot(on);
    if (act == 0) break;
    const int leader = __ffsll((long long)act) - 1;
    const u32 lead_bin = (u32)__builtin_amdgcn_readlane((int)bin, leader);
    const u64 grp = __ballot(on && bin == lead_bin);
    if (__popcll(grp) < 4) break;  // mixed bins: plain atomics below
    u32 b = 0;
    if (lane == (u32)leader) b = atomicAdd(&s[lead_bin], (u32)__popcll(grp));
    b = (u32)__builtin_amdgcn_readlane((int)b, leader);
    if (on && bin == lead_bin) {
      old = b + (u32)__popcll(grp & ((1ull << lane) - 1ull));
      on = false;
    }
  }
  if (on) old = atomicAdd(&s[bin], 1u);
  return old;
}

// Whether the calling workgroup is the last of `total` to get here (*done starts at zero); if
// so, everything the others wrote to global memory before is visible to it.  One thread
// fences for its workgroup: a fence at device scope writes back the XCD's whole L2, and with
// one per wave the label scan of a 1M-node graph took 27 us instead of 16.
__device__ __forceinline__ bool last_workgroup(u32* done, u32 total) {
  __shared__ u32 s_last;
  __builtin_amdgcn_s_waitcnt(0);  // this wave's stores have reached L2
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    s_last = atomicAdd(done, 1u) == total - 1u ? 1u : 0u;
    __threadfence();
  }
  __syncthreads();
  return s_last != 0;
}

__device__ __forceinline__ u32 hash_slot(u32 key, u32 log2cap) {
  return (key * 0x9E3779B1u) >> (32 - log2cap);
}

}  // namespace cq
