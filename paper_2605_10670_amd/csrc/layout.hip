// dispatch_layout: route every (token, j) pair to a live replica slot, count
// pairs per slot, prefix-sum the counts into receive-buffer offsets and give
// every routed pair its row, rows of one slot ordered by ascending token.
//
// Paper: Fig. 7 (the dispatch path skips peers whose `active` is 0), Sec. 5.1
// (slot -> logical expert map and all locations of each logical expert),
// Sec. 3.2 (validity contract), Sec. 4.1 (contiguous per-expert receive
// buffers as in prior work).
//
// One to three launches, all tiny and latency-bound (the step's metadata is
// < 1 MB), so the design goal is a short chain of dependent memory round trips,
// not bandwidth.  Up to 64 ranks the one-launch forms and k_map_count issue all their
// global loads before their first wait; k_scan_position reads the count matrix
// behind its first barrier, k_position the tile prefixes behind its scan.
//   k_layout_small  (<= 512 tokens and 4096 pairs) everything in one launch, see there.
//   k_layout_once  (<= 16384 pairs) the same for larger batches, see there.
//   k_map_count  one workgroup per tile of <= 128 tokens of ONE source rank.
//                Placement CSR, active mask and the tile's router indices are
//                fetched with independent loads.  For every slot the kernel
//                records a count and a bitmap of the tile's tokens that hit it:
//                popcount of the bits below a token is that pair's stable rank
//                inside the tile.  No atomics on positions, so the order is
//                deterministic.
//   k_scan_position  (<= 64 tiles) one workgroup per tile.  Lane = slot; the
//                workgroup's wavefronts share the rows of the [tiles][P] count
//                matrix (coalesced) for the slot totals and the pairs of
//                earlier tiles; one wavefront scans the totals; row = slot
//                offset + pairs of earlier tiles + rank in tile.  Each
//                workgroup repeats the small scan rather than wait for another
//                kernel.
//   k_tile_prefix + k_position  (> 64 tiles) the tile prefixes are computed once
//                by a few workgroups, then a wide grid computes the rows.
// Measured (a layout in a graph of 40; 32 ranks x 9 slots, top-8): T = 1024 / 4096 / 16384 in tiles
// 7.7 / 8.4 / 13.0 us; 9.7 / 10.5 / 14.3 while the live replicas were compacted per expert in
// LDS, the repeat check read LDS, counts were popcounts over the bitmaps, the scan took two
// barriers and half of k_scan_position's threads loaded the whole matrix.
#include <type_traits>

#include "eep_internal.hpp"
#include "rows.hpp"

namespace eep {

constexpr int kMapThreads = 1024;
constexpr int kPosThreads = 256;

// Tile b covers tokens [t0, t0 + ntok) of source rank b / tiles_per_rank; the
// last tile of a rank may be shorter, and no tile crosses into the next rank.
struct TileRange {
  int src_rank, sub_tile, t0, ntok;
};
__device__ inline TileRange tile_range(int b, int tokens_per_rank, int tiles_per_rank,
                                       int tile_tokens) {
  TileRange r;
  r.src_rank = b / tiles_per_rank;
  r.sub_tile = b - r.src_rank * tiles_per_rank;
  r.t0 = r.src_rank * tokens_per_rank + r.sub_tile * tile_tokens;
  int t1 = r.t0 + tile_tokens;
  const int rank_end = (r.src_rank + 1) * tokens_per_rank;
  if (t1 > rank_end) t1 = rank_end;
  r.ntok = t1 > r.t0 ? t1 - r.t0 : 0;
  return r;
}

// ---------------------------------------------------------------------------
// Routing tables in LDS, shared by the kernels that map pairs to slots.  What
// bounds those kernels is the chain of dependent round trips, so the tables
// take one: every global load is issued before the first wait, the active mask
// becomes a wave-wide ballot instead of an LDS array (R <= 64), and instead of
// a compacted list of live replicas per expert there is one bit per entry of
// the replica lists (`alive`), from which a pair counts and picks its replica.
// ---------------------------------------------------------------------------
struct RouteTables {
  int32_t* off;     // [E+1] replica-list starts (CSR)
  int32_t* list;    // [P] replica lists, canonical order
  uint32_t* alive;  // [alive_words(P)] bit q: the replica in list[q] is on an active rank
};

// Bits are written 64 at a time; a pair whose expert's list starts at o <= P reads the words
// o / 32 and o / 32 + 1, so two more words follow.
__host__ __device__ inline int alive_words(int P) { return (P + 63) / 64 * 2 + 2; }
__host__ __device__ inline size_t route_table_ints(int E, int P, int R) {
  return (size_t)(E + 1) + P + alive_words(P) + mask_words(R);
}

// Rank that owns slot p: p / S with inv_S = 1.0f / S.  (p + 0.5) / S is at least 0.5 / S away
// from an integer and the float result at most (P / S) * 2^-23 off, so it is exact for all
// P < 2^22; the library's limit is 2^20.
__device__ __forceinline__ int rank_of_slot(int p, float inv_S) {
  return (int)(((float)p + 0.5f) * inv_S);
}

// Fills the tables at `lds` (route_table_ints of it) with the whole workgroup of nt threads, in
// two steps: `fetch` at the very start of a kernel, so that its loads are out before anything is
// waited for, and `fill`; the caller's next barrier makes the tables readable.  LARGE: more than 64 ranks
// (the mask goes through LDS, which takes one barrier here) or tables of more than nt words.
// `agree` may replace the mask: it is called with the 64-bit mask, or (LARGE) with its words in LDS, and the
// whole workgroup.
struct OwnMask {
  __device__ __forceinline__ uint64_t operator()(uint64_t mask) const { return mask; }
  __device__ __forceinline__ void operator()(uint32_t*) const {}
};
inline bool large_tables(int E, int P, int R, int threads) { return R > 64 || P > threads || E >= threads; }
template <bool LARGE>
struct RouteTableLoad {
  const int32_t *l2p_off, *l2p_list, *active;
  int E, R, P, nt, a, p, o;
  __device__ __forceinline__ void fetch() {
    const int tid = threadIdx.x, lane = tid & 63;
    a = active[lane < R ? lane : R - 1];
    p = l2p_list[tid < P ? tid : P - 1];
    o = l2p_off[tid < E ? tid : E];
  }
  template <class Agree = OwnMask>
  __device__ __forceinline__ RouteTables fill(int32_t* lds, float inv_S, Agree agree = Agree()) const {
    RouteTables rt;
    rt.off = lds;
    rt.list = rt.off + (E + 1);
    rt.alive = (uint32_t*)(rt.list + P);
    const int tid = threadIdx.x, lane = tid & 63;
    if constexpr (!LARGE) {
      if (tid <= E) rt.off[tid] = o;
      const uint64_t mask = agree(__ballot(lane < R && a != 0));
      const bool slot = tid < P && p >= 0;
      if (tid < P) rt.list[tid] = p;
      const uint64_t bits = __ballot(slot && ((mask >> (rank_of_slot(p, inv_S) & 63)) & 1));
      if (lane == 0 && tid < P) {
        rt.alive[tid >> 5] = (uint32_t)bits;
        rt.alive[(tid >> 5) + 1] = (uint32_t)(bits >> 32);
      }
    } else {
      uint32_t* mask = rt.alive + alive_words(P);
#pragma nounroll
      for (int r = tid; r - lane < R; r += nt) {
        const uint64_t bits = __ballot(r < R && active[r] != 0);
        if (lane == 0) {
          mask[r >> 5] = (uint32_t)bits;
          if ((r >> 5) + 1 < mask_words(R)) mask[(r >> 5) + 1] = (uint32_t)(bits >> 32);
        }
      }
#pragma nounroll
      for (int i = tid; i <= E; i += nt) rt.off[i] = i == tid ? o : l2p_off[i];
      __syncthreads();
      agree(mask);
#pragma nounroll
      for (int q = tid; q - lane < P; q += nt) {  // whole wavefronts, for the ballot
        const int v = q == tid ? p : q < P ? l2p_list[q] : -1;
        if (q < P) rt.list[q] = v;
        const bool slot = q < P && (unsigned)v < (unsigned)P;  // (past the last list a caller may leave anything)
        const int r = slot ? rank_of_slot(v, inv_S) : 0;
        const uint64_t bits = __ballot(slot && ((mask[r >> 5] >> (r & 31)) & 1));
        if (lane == 0) {
          rt.alive[(q >> 5)] = (uint32_t)bits;
          rt.alive[(q >> 5) + 1] = (uint32_t)(bits >> 32);
        }
      }
    }
    if (tid < 2) rt.alive[alive_words(P) - 1 - tid] = 0;
    return rt;
  }
};

// The live replica that serves token t's pair with expert e (in [0, E)), or -1.
__device__ __forceinline__ int pick_slot(const RouteTables& rt, int e, int t, int policy) {
  const int o = rt.off[e], m = rt.off[e + 1] - o;  // m replicas, dead ones included
  if (m <= 32) {
    // bits o .. o + 31 of `alive`, the first m of them the expert's
    const uint64_t two = (uint64_t)rt.alive[(o >> 5) + 1] << 32 | rt.alive[o >> 5];
    uint32_t bits = (uint32_t)(two >> (o & 31)) & (uint32_t)((1ull << m) - 1);
    if (bits == 0) return -1;
    const int n = __popc(bits);
    int sel = (policy == EEP_FIRST_LIVE || n == 1) ? 0 : n == 2 ? t & 1 : t % n;
    for (; sel > 0; --sel) bits &= bits - 1;
    return rt.list[o + __ffs(bits) - 1];
  }
  int n = 0;
  for (int q = o; q < o + m; ++q) n += (rt.alive[q >> 5] >> (q & 31)) & 1;
  if (n == 0) return -1;
  int sel = policy == EEP_FIRST_LIVE ? 0 : t % n;
  int q = o;
  for (;; ++q)
    if ((rt.alive[q >> 5] >> (q & 31)) & 1) {
      if (sel == 0) break;
      --sel;
    }
  return rt.list[q];
}

// Does pair j of a token repeat an earlier expert of it?  Pairs are laid out token by token,
// one per lane from a multiple of k on, so for k a power of two <= 16 a token's pairs lie in
// one DPP row and the earlier ones are reached without LDS; other k read the token's
// indices (`token_idx`, k of them).
template <int SHR>
__device__ __forceinline__ bool earlier_lane_equals(int e, int j) {
  const int v = __builtin_amdgcn_update_dpp(-1, e, 0x110 + SHR, 0xf, 0xf, false);  // row_shr:SHR
  return j >= SHR && v == e;
}
// x ^ the value CTRL away, lane to lane inside groups of 8
template <int CTRL>
__device__ __forceinline__ uint32_t lane_xor(int from, int e) {
  return (uint32_t)(__builtin_amdgcn_update_dpp(0, from, CTRL, 0xf, 0xf, false) ^ e);
}
template <int KC>
__device__ __forceinline__ bool repeats_earlier(int e, int j, const int32_t* token_idx) {
  bool r = false;
  if constexpr (KC == 0) {
    // eight and then four at a time, so that their latencies overlap (up to three words behind the
    // token's are read): top-32, 64 tokens 6.6 us, four at a time 7.1
    const auto look = [&](int jj, auto n) {
      constexpr int N = decltype(n)::value;
      int v[N];
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = token_idx[jj + u];
#pragma unroll
      for (int u = 0; u < N; ++u) r |= jj + u < j && v[u] == e;
    };
    int jj = 0;
#pragma nounroll
    for (; jj + 4 < j; jj += 8) look(jj, std::integral_constant<int, 8>());
    if (jj < j) look(jj, std::integral_constant<int, 4>());
  } else if constexpr (KC > 1) {
    static_assert(KC == 2 || KC == 4 || KC == 8, "pairs of a token share a DPP row");
    // first whether any two of the token's lanes are equal (quad_perm 1032, 2301, 3210; the other
    // quad by way of row_half_mirror), which is rarely so
    uint32_t least = lane_xor<0xB1>(e, e);
    if constexpr (KC > 2) least = min(least, min(lane_xor<0x4E>(e, e), lane_xor<0x1B>(e, e)));
    if constexpr (KC > 4) {
      const int m = __builtin_amdgcn_update_dpp(0, e, 0x141, 0xf, 0xf, false);
      least = min(least, min((uint32_t)(m ^ e), lane_xor<0xB1>(m, e)));
      least = min(least, min(lane_xor<0x4E>(m, e), lane_xor<0x1B>(m, e)));
    }
    if (__builtin_expect(__any(least == 0), 0)) {
      r = earlier_lane_equals<1>(e, j);
      if constexpr (KC > 2) {
        r |= earlier_lane_equals<2>(e, j);
        r |= earlier_lane_equals<3>(e, j);
      }
      if constexpr (KC > 4) {
        r |= earlier_lane_equals<4>(e, j);
        r |= earlier_lane_equals<5>(e, j);
        r |= earlier_lane_equals<6>(e, j);
        r |= earlier_lane_equals<7>(e, j);
      }
    }
  }
  return r;
}

// A token can hit a slot at most once: its k logical experts are distinct
// (repeats are masked) and a slot holds one logical expert.  So one bit per
// (slot, token of the tile) is enough: popcount of the bits below a token is
// its stable rank in the slot.  The slot's count is kept beside the bitmap, so
// that nobody has to walk the words for it.
constexpr int kMaxPairsPerThread = kTileTokens * kMaxTopk / kMapThreads;

// Maps this thread's pairs tid, tid + NT, ... (NT threads) of a batch of `npairs` (first token t0):
// slots to slot[] (-1: not routed), token bits to s_bm
// ([P][stride], zeroed), counts to s_count (zeroed), dropped pairs to s_drop {uncovered, masked}
// (zeroed).  my_e holds the router indices already loaded; s_idx the same in LDS when KC == 0.  Slots of
// the pairs [own_lo, own_hi) are written to slot_of.
template <int KC, int U, int NT = kMapThreads>
__device__ __forceinline__ void map_pairs(const RouteTables& rt, const int (&my_e)[U],
                                          const int32_t* s_idx, int (&slot)[U], uint32_t* s_bm,
                                          int stride, int32_t* s_count, int32_t* s_drop, int npairs,
                                          int k, int E, int t0, int policy, int own_lo,
                                          int own_hi, int32_t* __restrict__ slot_of) {
  const int wave0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = threadIdx.x + u * NT;
    slot[u] = -1;
    if (wave0 + u * NT >= npairs) break;  // a wavefront without pairs stays out of the others' way
    const int tl = i / k, j = i - tl * k;
    const int e = my_e[u];
    const bool repeated = repeats_earlier<KC>(e, j, KC == 0 && i < npairs ? s_idx + tl * k : s_idx);
    if (i < npairs) {
      int p = -1;
      if ((unsigned)e >= (unsigned)E || repeated) {
        atomicAdd(&s_drop[1], 1);
      } else {
        p = pick_slot(rt, e, t0 + tl, policy);
        if (p < 0) {
          atomicAdd(&s_drop[0], 1);
        } else {
          atomicOr(&s_bm[p * stride + (tl >> 5)], 1u << (tl & 31));
          atomicAdd(&s_count[p], 1);
        }
      }
      slot[u] = p;
      if (i >= own_lo && i < own_hi) slot_of[i] = p;
    }
  }
}

// Stable rank of token tl in a slot: tokens before it in the slot's bitmap.  Words are read four
// at a time, so that their LDS latencies overlap; up to three of them lie behind the token's
// own word and are not counted (they may belong to the next slot, or to the array behind
// the bitmaps: the caller's LDS goes on for at least three words).
__device__ __forceinline__ int rank_in_slot(const uint32_t* bm, int tl) {
  const int tw = tl >> 5;
  int r = __popc(bm[tw] & ((1u << (tl & 31)) - 1u));
  for (int w = 0; w < tw; w += 4) {
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = bm[w + u];
#pragma unroll
    for (int u = 0; u < 4; ++u) r += w + u < tw ? __popc(v[u]) : 0;
  }
  return r;
}

// LDS ints of the map kernel for a tile: tables, counts, bitmaps, and the router indices
// where k is not handled lane to lane.
inline size_t map_lds_ints(int E, int P, int R, int tile_tokens, int k) {
  return route_table_ints(E, P, R) + P + (size_t)P * kBitmapWords + (size_t)tile_tokens * k;
}

template <int KC, int U, bool LARGE>  // KC = compile-time k (power of two) or 0 for any k
__global__ __launch_bounds__(kMapThreads) void k_map_count(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ l2p_off,
    const int32_t* __restrict__ l2p_list, const int32_t* __restrict__ active, int k_rt,
    int tokens_per_rank, int tiles_per_rank, int tile_tokens, int E, int P, int R, float inv_S,
    int policy, int32_t* __restrict__ slot_of, int32_t* __restrict__ rank_in_tile,
    int32_t* __restrict__ cnt_tile, int32_t* __restrict__ blk_unc,
    int32_t* __restrict__ blk_msk) {
  const int k = KC > 0 ? KC : k_rt;
  extern __shared__ int32_t smem[];
  int32_t* s_count = smem;                       // [P] pairs of the tile per slot
  uint32_t* s_bm = (uint32_t*)(s_count + P);     // [P][kBitmapWords]
  int32_t* s_idx = (int32_t*)(s_bm + P * kBitmapWords);  // [tile_tokens*k], KC == 0 only
  int32_t* s_tab = s_idx + (KC == 0 ? tile_tokens * k : 0);
  __shared__ int32_t s_drop[2];

  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  const TileRange tr = tile_range(b, tokens_per_rank, tiles_per_rank, tile_tokens);
  const int npairs = tr.ntok * k;
  const int64_t g0 = (int64_t)tr.t0 * k;

  int my_e[U], slot[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = tid + u * kMapThreads;
    my_e[u] = i < npairs ? topk_idx[g0 + i] : -1;
  }
  RouteTableLoad<LARGE> tables = {l2p_off, l2p_list, active, E, R, P, kMapThreads};
  tables.fetch();
#pragma nounroll
  for (int i = tid; i < P * (kBitmapWords + 1); i += kMapThreads) s_count[i] = 0;  // and s_bm
  if (tid < 2) s_drop[tid] = 0;
  const RouteTables rt = tables.fill(s_tab, inv_S);
  if constexpr (KC == 0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (tid + u * kMapThreads < npairs) s_idx[tid + u * kMapThreads] = my_e[u];
  }
  __syncthreads();
  map_pairs<KC, U>(rt, my_e, s_idx, slot, s_bm, kBitmapWords, s_count, s_drop, npairs, k, E, tr.t0,
                   policy, 0, npairs, slot_of + g0);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = tid + u * kMapThreads;
    if (i < npairs)
      rank_in_tile[g0 + i] = slot[u] >= 0 ? rank_in_slot(&s_bm[slot[u] * kBitmapWords], i / k) : -1;
  }
  for (int p = tid; p < P; p += kMapThreads) cnt_tile[(int64_t)b * P + p] = s_count[p];
  if (tid == 0) {
    blk_unc[b] = s_drop[0];
    blk_msk[b] = s_drop[1];
  }
}

// Inclusive scan across the 64 lanes of a wavefront, in DPP (no LDS round trips).
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
  return v;
}

// Exclusive scan of value(0..n) into s_offset[0..n] by ONE wavefront, 64 values at a time
// and kScanChunks such groups at once (their loads and scans are independent; only the running
// sum is a chain).  The caller's next barrier makes the result readable.
constexpr int kScanChunks = 5;
template <class Value>
__device__ __forceinline__ void wave_exclusive_scan(Value value, int32_t* s_offset, int n) {
  const int lane = threadIdx.x & 63;
  int run = 0;
  for (int c0 = 0; c0 < n; c0 += 64 * kScanChunks) {
    int v[kScanChunks], incl[kScanChunks];
#pragma unroll
    for (int c = 0; c < kScanChunks; ++c) {
      const int p = c0 + c * 64 + lane;
      v[c] = p < n ? value(p) : 0;
    }
#pragma unroll
    for (int c = 0; c < kScanChunks; ++c) incl[c] = wave_inclusive_scan(v[c]);
#pragma unroll
    for (int c = 0; c < kScanChunks; ++c) {
      const int p = c0 + c * 64 + lane;
      if (p < n) s_offset[p] = run + incl[c] - v[c];
      run += __builtin_amdgcn_readlane(incl[c], 63);
    }
  }
  if (lane == 0) s_offset[n] = run;
}

// Exclusive scan of the slots' totals into s_offset[0..P]: the wavefronts, the last one first, take
// 64 slots each and add up what lies ahead of these for themselves, so that nothing has to be
// exchanged.  The caller's next barrier makes the result readable.
template <class Total>
__device__ __forceinline__ void scan_totals(Total total, int32_t* s_offset, int P, int wave,
                                            int waves) {
  const int lane = threadIdx.x & 63, chunks = (P >> 6) + 1;
#pragma nounroll
  for (int c = waves - 1 - wave; c < chunks; c += waves) {
    int ahead = 0;
#pragma unroll 4
    for (int i = 0; i < c; ++i) ahead += total(i * 64 + lane);
    const int p = c * 64 + lane, v = p < P ? total(p) : 0;
    const int incl = wave_inclusive_scan(v);
    ahead = __builtin_amdgcn_readlane(wave_inclusive_scan(ahead), 63);
    if (p <= P) s_offset[p] = ahead + incl - v;
  }
}

// Per-step tables every consumer needs, written once by one workgroup
// (`count` may be null when another kernel has already written it).
__device__ inline void write_step_tables(int nt, const int32_t* s_offset,
                                         int dropped_unc, int dropped_msk, int version,
                                         int32_t* __restrict__ count, int32_t* __restrict__ offset,
                                         int32_t* __restrict__ rank_count,
                                         int32_t* __restrict__ rank_offset,
                                         int32_t* __restrict__ status,
                                         int32_t* __restrict__ step_epoch, int R, int S, int P) {
  const int tid = threadIdx.x;
#pragma nounroll
  for (int p = tid; p <= P; p += nt) {
    offset[p] = s_offset[p];
    if (count != nullptr && p < P) count[p] = s_offset[p + 1] - s_offset[p];
  }
#pragma nounroll
  for (int r = tid; r < R; r += nt) {
    rank_offset[r] = s_offset[r * S];
    rank_count[r] = s_offset[(r + 1) * S] - s_offset[r * S];
  }
  if (tid == 0) {
    rank_offset[R] = s_offset[P];
    status[0] = s_offset[P];
    status[1] = dropped_unc;
    status[2] = dropped_msk;
    status[3] = version;
    *step_epoch = *step_epoch + 1;  // one increment per step, on the device (graph replays too)
  }
}

// ---------------------------------------------------------------------------
// Few tiles (<= 64, the decode regime): scan and position fused.  Every
// workgroup (one per tile) re-derives what it needs from the [tiles][P] count
// matrix -- slot totals and the pairs of earlier tiles -- with lane = slot and
// the tiles shared between the wavefronts, so that a wavefront has one round of
// loads (three sets of wavefronts at 288 slots: 11 loads at 32 tiles, 22 in two
// rounds at 64).  Measured (T = 1024 / 4096 / 5976, whole layout): 12 loads per
// round 7.8 / 8.5 / 8.5 us, 8 7.9 / 8.5 / 8.1, 16 8.0 / 8.6 / 8.7; 512 threads 8.4 / 9.0 / 8.3.
// ---------------------------------------------------------------------------
constexpr int kFusedThreads = 1024;
constexpr int kFusedWaves = kFusedThreads / 64;
constexpr int kFusedPairs = 2048 / kFusedThreads;  // pairs of the tile kept in registers per thread
constexpr int kFusedBatch = 12;   // count-matrix rows fetched per round
constexpr int kTileBatch = 32;    // count-matrix rows k_tile_prefix fetches per round

template <int KC>
__global__ __launch_bounds__(kFusedThreads) void k_scan_position(
    const int32_t* __restrict__ cnt_tile, const int32_t* __restrict__ slot_of,
    int32_t* __restrict__ row_of, int P, int num_tiles, int k_rt, int tokens_per_rank,
    int tiles_per_rank, int tile_tokens, const int32_t* __restrict__ blk_unc,
    const int32_t* __restrict__ blk_msk, const int32_t* __restrict__ tbl_version,
    const int32_t* __restrict__ mem_version, int R, int S, int32_t* __restrict__ src_of,
    int32_t* __restrict__ count, int32_t* __restrict__ offset, int32_t* __restrict__ rank_count,
    int32_t* __restrict__ rank_offset, int32_t* __restrict__ cnt_src,
    int32_t* __restrict__ status, int32_t* __restrict__ step_epoch) {
  const int k = KC > 0 ? KC : k_rt;
  extern __shared__ int32_t smem[];
  int32_t* s_count = smem;           // [P]   pairs per slot, all tiles
  int32_t* s_offset = s_count + P;   // [P+1] exclusive scan of s_count
  int32_t* s_pre = s_offset + P + 1; // [P]   pairs per slot in tiles before this one
  __shared__ int32_t s_drop[2];
  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  const TileRange tr = tile_range(b, tokens_per_rank, tiles_per_rank, tile_tokens);
  const int src_rank = tr.src_rank, sub_tile = tr.sub_tile;
  const int npairs = tr.ntok * k;
  const int g0 = tr.t0 * k;
  const int first = src_rank * tiles_per_rank;  // tiles [first, first + tiles_per_rank) share
                                                // this tile's source rank

  int my_slot[kFusedPairs], my_rank[kFusedPairs];
#pragma unroll
  for (int u = 0; u < kFusedPairs; ++u) {
    int i = tid + u * kFusedThreads;
    my_slot[u] = i < npairs ? slot_of[g0 + i] : -1;
    my_rank[u] = i < npairs ? row_of[g0 + i] : 0;  // rank inside the tile
  }
  int du = 0, dm = 0, version = 0;
  if (b == 0) {
    for (int i = tid; i < num_tiles; i += kFusedThreads) {
      du += blk_unc[i];
      dm += blk_msk[i];
    }
    if (tid == 0) version = *tbl_version + *mem_version;
  }
  if (tid < 2) s_drop[tid] = 0;
  for (int p = tid; p < P; p += kFusedThreads) s_count[p] = s_pre[p] = 0;
  // Wavefronts take 64 slots each, and as many sets of wavefronts as fit share the tiles; the
  // sets' sums meet in LDS.
  const int slot_waves = (P + 63) / 64;
  const int sets = kFusedWaves > slot_waves ? kFusedWaves / slot_waves : 1;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __syncthreads();
  for (int w = wave; w < sets * slot_waves; w += kFusedWaves) {
    const int set = w / slot_waves;
    const int p = (w - set * slot_waves) * 64 + (tid & 63);
    int total = 0, before = 0;
    for (int tb = set; tb < num_tiles; tb += sets * kFusedBatch) {
      int v[kFusedBatch];
#pragma unroll
      for (int u = 0; u < kFusedBatch; ++u) {
        const int tile = tb + u * sets;
        v[u] = tile < num_tiles && p < P ? cnt_tile[(int64_t)tile * P + p] : 0;
      }
#pragma unroll
      for (int u = 0; u < kFusedBatch; ++u) {
        total += v[u];
        before += tb + u * sets < b ? v[u] : 0;
      }
    }
    if (p < P) {
      atomicAdd(&s_count[p], total);
      atomicAdd(&s_pre[p], before);
    }
  }
  if (sub_tile == 0)  // pairs per (source rank, slot): the source rank's own tiles
    for (int p = tid; p < P; p += kFusedThreads) {
      int part = 0;
      for (int t = first; t < first + tiles_per_rank; ++t) part += cnt_tile[(int64_t)t * P + p];
      cnt_src[(int64_t)src_rank * P + p] = part;
    }
  __syncthreads();
  if (du) atomicAdd(&s_drop[0], du);  // zeroed before the barrier, read after the scan's barriers
  if (dm) atomicAdd(&s_drop[1], dm);
  if (tid < 64) wave_exclusive_scan([=](int p) { return s_count[p]; }, s_offset, P);
  __syncthreads();

  const int N = s_offset[P];
#pragma unroll
  for (int u = 0; u < kFusedPairs; ++u) {
    int i = tid + u * kFusedThreads;
    if (i < npairs) {
      int p = my_slot[u];
      int row = -1;
      if (p >= 0) {
        row = s_offset[p] + s_pre[p] + my_rank[u];
        src_of[row] = g0 + i;
      }
      row_of[g0 + i] = row;
      if (g0 + i >= N) src_of[g0 + i] = -1;  // rows past the last routed pair
    }
  }
  if (b == 0)
    write_step_tables(kFusedThreads, s_offset, s_drop[0], s_drop[1], version, count,
                                     offset, rank_count, rank_offset, status, step_epoch, R, S, P);
}

// ---------------------------------------------------------------------------
// Small batches (at most 512 tokens and 4096 pairs) in ONE launch with a token bitmap per slot that spans
// the batch, a pair to a lane.  Bound by latency: the launch (1.9 us for an empty kernel), one round of
// global loads, LDS round trips, and stores.  Every workgroup maps ALL pairs (1 to 4 per thread, each
// keeps the whole count and offset table) and then writes its eighth of the results, so no
// workgroup waits for another; one alone spent 1.4 to 2.8 us on storing, mostly the [R][P] matrix of pairs per
// (source rank, slot).
//
// Where k_layout_once below could do it too, this takes at most a pair to a thread (kFewPairs), with a compile-time k.
// Measured (a layout in a graph of 40; 32 ranks x 9 slots, in brackets that one): top-8, T = 32 / 64 / 128 3.55 / 3.6
// / 3.7 us (4.1 each), T = 192 / 256 / 512 4.3 / 4.6 / 5.8 (4.2 / 4.3 / 4.5); top-4, T = 64 / 128 / 256 / 512 3.6 / 3.6 /
// 3.8 / 4.5 (3.8 / 3.8 / 3.9 / 4.0); top-2, T = 64 / 128 / 512 3.5 / 3.6 / 3.8 (3.7 / 3.8 / 3.8); top-1, T = 512 3.65 (3.65);
// without a compile-time k, top-6, T = 32 / 64 / 128 4.0 / 4.05 / 4.2 (4.0 each); 64 ranks, top-8, T = 64 / 128 / 256
// 3.9 / 4.1 / 5.0 (4.9 / 4.9 / 5.0); 24 ranks x 17 slots, T = 120, top-2 3.9 (3.8), top-8 4.0 (4.3); 48 x 10, top-2,
// T = 144 3.9 (4.15); 6 x 5, top-1, T = 420, five replicas 3.3 (3.9).
// Beyond these it takes more than top-10, and tables that do not fit there (8 ranks x 265 slots, T = 32: 7.6 us, in
// tiles 12.6).  With the scan done by one wavefront, and the source ranks' counts by the first workgroups'
// wavefronts alone, it took 0.05 to 0.5 us more, and most with more than 320 slots (64 ranks 4.4 / 4.5, 24 x 17 4.5).
//
// The eight results fit together only if all eight workgroups saw one mask.  An
// instance of one context keeps its mask still while a layout runs: only its own
// later calls on the stream change it.  With several contexts another one's combine
// may drop a rank, or another one's caller may update the mask, at any moment.  So
// there ONE workgroup does it all (each entry of the replica lists is found live or
// dead once, and every pair, count and row follows from that), up to the size from
// which the tiled path, where each pair is mapped once, is as fast: T = 32 / 128 / 256 / 384
// 4.0 / 4.4 / 5.6 / 7.2 us, in tiles 7.5.  Tiles are what comes next without a context, where nobody can agree on a
// mask; the limit is the same with several, where k_layout_once comes next.  (That one is the faster already from about 2048 pairs
// on, with many slots earlier and with few later, a layout in a graph of 40, one workgroup / agreement: 32 ranks x 9 slots, top-8, T = 160 / 224 / 256 /
// 320 / 384 4.8 / 5.1 / 5.5 / 6.25 / 7.05 and 5.05 / 5.3 / 4.9 / 5.1 / 5.3 us; 64 x 9, T = 192 / 384 7.8 / 10.1 and 5.5 / 5.6; 4 x 6, T = 256 / 320 / 384
// 4.3 / 4.9 / 5.2 and 4.8 / 4.9 / 4.95.)  The launch
// decides by the number of contexts; a launch captured while there was one is
// overruled by the word behind the membership version, which says that there are more.
// ---------------------------------------------------------------------------
constexpr int kSmallBlocks = 8;
constexpr int kSmallTokens = 512;
constexpr int kSmallPairsPerThread = 4;
constexpr int kSmallPairs = kMapThreads * kSmallPairsPerThread;
constexpr int kSoloTokens = 384;  // the limits for one workgroup
constexpr int kSoloPairs = kMapThreads * 3;
constexpr int kFewPairs = kMapThreads;  // up to here not for k_layout_once
constexpr uint32_t kSoloBit = 1u << 31;

__device__ __forceinline__ int vector_load(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Row stride of token bitmaps in words; odd, so that lanes on different slots reading
// the same word index hit different banks.
__host__ __device__ inline int token_stride(int tokens) { return ((tokens + 31) / 32) | 1; }
inline size_t small_lds_bytes(int E, int P, int R, int T, int k) {
  return sizeof(int32_t) * (route_table_ints(E, P, R) + P + (P + 1) +
                            (size_t)P * token_stride(T) + (size_t)T * k);
}

// cnt[p] = tokens [lo, hi) in the bitmap of slot p, for the kSrcChunks * 64 slots from p0 on;
// lo < hi are the same for the whole wavefront.  The slots' words are read side by side, so
// that the LDS latencies overlap.
template <int kSrcChunks>
__device__ __forceinline__ void store_src_counts(const uint32_t* s_bm, int stride, int p0, int P,
                                                 int lo, int hi, int32_t* __restrict__ cnt) {
  const int w0 = lo >> 5, w1 = (hi - 1) >> 5;
  int c[kSrcChunks] = {};
  for (int w = w0; w <= w1; ++w) {
    uint32_t m = ~0u;
    if (w == w0) m &= ~0u << (lo & 31);
    if (w == w1) m &= ~0u >> (31 - ((hi - 1) & 31));
    uint32_t v[kSrcChunks];
#pragma unroll
    for (int u = 0; u < kSrcChunks; ++u) {
      const int p = p0 + u * 64 + (int)(threadIdx.x & 63);
      v[u] = s_bm[(p < P ? p : P - 1) * stride + w];
    }
#pragma unroll
    for (int u = 0; u < kSrcChunks; ++u) c[u] += __popc(v[u] & m);
  }
#pragma unroll
  for (int u = 0; u < kSrcChunks; ++u) {
    const int p = p0 + u * 64 + (int)(threadIdx.x & 63);
    if (p < P) cnt[p] = c[u];
  }
}

template <int KC, int U, bool LARGE>
__global__ __launch_bounds__(kMapThreads) void k_layout_small(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ l2p_off,
    const int32_t* __restrict__ l2p_list, const int32_t* __restrict__ active,
    const int32_t* __restrict__ mem_version, uint32_t T_k, int E, int P, int R, float inv_S,
    const int32_t* __restrict__ tbl_version, int policy, int tokens_per_rank, int S,
    int32_t* __restrict__ slot_of, int32_t* __restrict__ row_of, int32_t* __restrict__ src_of,
    int32_t* __restrict__ count, int32_t* __restrict__ offset, int32_t* __restrict__ rank_count,
    int32_t* __restrict__ rank_offset, int32_t* __restrict__ cnt_src,
    int32_t* __restrict__ status, int32_t* __restrict__ step_epoch) {
  const int T = T_k & 0xffff, k = KC > 0 ? KC : T_k >> 16 & 0xff;  // in one preloaded word
  const int npairs = T * k;
  const int stride = token_stride(T);
  extern __shared__ int32_t smem[];
  int32_t* s_count = smem;                        // [P] pairs per slot
  uint32_t* s_bm = (uint32_t*)(s_count + P);      // [P][stride] token bitmap per slot
  int32_t* s_offset = (int32_t*)(s_bm + P * stride);  // [P+1] exclusive scan of s_count
  int32_t* s_idx = s_offset + P + 1;              // [T*k] router indices, KC == 0 only
  int32_t* s_tab = s_idx + (KC == 0 ? npairs : 0);
  __shared__ int32_t s_drop[2];
  const int tid = threadIdx.x;

  // every global read of this kernel is issued here, none depends on another
  int my_e[U], slot[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = tid + u * kMapThreads;
    my_e[u] = i < npairs ? topk_idx[i] : -1;
  }
  const int version = blockIdx.x == 0 && tid == 0 ? *tbl_version + *mem_version : 0;
  // several contexts in the instance: the first workgroup does it all.  (A vector load: a scalar one
  // would be waited for together with every kernel argument.)
  const int several_v = vector_load(&mem_version[1]);
  RouteTableLoad<LARGE> tables = {l2p_off, l2p_list, active, E, R, P, kMapThreads};
  tables.fetch();
#pragma nounroll
  for (int i = tid; i < P * (stride + 1); i += kMapThreads) s_count[i] = 0;  // and s_bm
  if (tid < 2) s_drop[tid] = 0;
  const RouteTables rt = tables.fill(s_tab, inv_S);
  if constexpr (KC == 0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (tid + u * kMapThreads < npairs) s_idx[tid + u * kMapThreads] = my_e[u];
  }
  // the pairs [own_lo, own_hi) whose results this workgroup writes, and as which of how many; with
  // `solo` the first one's are all, the others go along and write nothing
  const bool solo = __builtin_amdgcn_readfirstlane(several_v) != 0 || (T_k & kSoloBit) != 0;
  const int blocks = solo ? 1 : kSmallBlocks, block = solo && blockIdx.x > 0 ? R : blockIdx.x;
  const int share = ((npairs + kSmallBlocks - 1) / kSmallBlocks + 63) & ~63;
  const int own_lo = solo ? (blockIdx.x > 0 ? npairs : 0) : blockIdx.x * share;
  const int own_hi = solo || own_lo + share > npairs ? npairs : own_lo + share;
  __syncthreads();
  map_pairs<KC, U>(rt, my_e, s_idx, slot, s_bm, stride, s_count, s_drop, npairs, k, E, 0, policy, own_lo,
                   own_hi, slot_of);
  __syncthreads();

  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  scan_totals([=](int p) { return s_count[p]; }, s_offset, P, wave, kMapThreads / 64);
  __syncthreads();

  const int N = s_offset[P];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = tid + u * kMapThreads;
    if (i >= own_lo && i < own_hi) {
      const int p = slot[u];
      int row = -1;
      if (p >= 0) {
        row = s_offset[p] + rank_in_slot(&s_bm[p * stride], i / k);
        src_of[row] = i;
      }
      row_of[i] = row;
      if (i >= N) src_of[i] = -1;  // rows past the last routed pair
    }
  }
  // pairs per (source rank, slot): the tokens of a source rank are a bit range; wavefronts
  // take source ranks, the workgroups in turn, lanes slots, five sets of 64 at once where there are more than one
  for (int b = wave * blocks + block; b < R; b += blocks * (kMapThreads / 64)) {
    const int lo = b * tokens_per_rank, hi = lo + tokens_per_rank;
    int32_t* cnt = cnt_src + (int64_t)b * P;
    if (P <= 64)
      store_src_counts<1>(s_bm, stride, 0, P, lo, hi, cnt);
    else
      for (int p0 = 0; p0 < P; p0 += 320) store_src_counts<5>(s_bm, stride, p0, P, lo, hi, cnt);
  }
  if (blockIdx.x == 0)
    write_step_tables(kMapThreads, s_offset, s_drop[0], s_drop[1], version, count, offset, rank_count,
                      rank_offset, status, step_epoch, R, S, P);
}

// ---------------------------------------------------------------------------
// The whole layout in ONE launch, for batches up to 16384 pairs.  A workgroup owns a
// share of the tokens.  It counts the pairs per slot of ALL tokens,
// those ahead of its share, its own and those behind it apart, so it needs nothing from
// the others; then it places its own.  Bound by latency and by instructions: the launch
// (1.9 us for an empty kernel), one round of global loads, LDS round trips, and, as every
// workgroup maps all pairs, the instructions per pair.  Hence a lane takes a whole token,
// whose indices it compares in registers, the routing of an expert is one word that is
// prepared once (`build_entries`), pairs without a slot have sinks to be counted in instead
// of a branch, and what does not wait for the scan stands between its barriers.
//
// Measured (a layout in a graph of 40; 32 ranks x 9 slots, top-8), in brackets k_layout_small, and beyond 512
// tokens tiles: T = 256 / 512 4.3 / 4.5 us (4.6 / 5.8), 1024 / 1536 / 2048 5.1 / 5.5 / 6.0 (7.6 / 7.8 / 7.9), 3072 / 4096
// 7.3 / 8.3 (8.0 / 8.3); with a Zipf router, whose hot slots' counts are one LDS word for many lanes, 2048 / 3072 / 4096
// 6.4 / 7.9 / 9.1 (7.8 / 7.9 / 8.1).  T = 1024 of 64 ranks x 9 slots 5.6 (12.0), top-2 of 32 ranks 3.95 (7.4), T = 768 of 24
// ranks, top-6, 4.4 (7.8).  So up to 16384 pairs.  Shares of about 64 tokens, whole
// source ranks or, where a rank has at least 768 pairs, a part of one, whose first then also counts the
// rank's other tokens for the rank's totals: 8 ranks, T = 1024 / 2048 5.0 / 6.2 (whole ranks 5.5 / 7.2; tiles
// 7.9 / 8.1), 2 ranks, T = 512 / 1024 / 2048 4.4 / 5.3 / 7.3 (5.5 / 8.7 / 14.7; 5.9 / 7.2 / 7.8), 4 ranks, top-3,
// T = 1024 3.9 (4.5; 7.2); with fewer pairs it costs as much as it gives (32 ranks, top-2, T = 4096, 256
// pairs to a rank: 5.0 in parts, 4.8).  512 threads, 1024 for more than 1024 tokens (T = 256 / 512 / 1024: 4.25 / 4.5 /
// 5.1 with 512, 4.35 / 4.6 / 5.0 with 1024).
//
// What no ordinary router gives: 2048 tokens, 90 % of them without an expert (-1) 6.2 us (17.3 with one sink for all,
// tiles 8.7), half of all pairs without one 6.4 (11.9; 8.8), all tokens alike 6.5 (17.4 lane by lane; 7.7), one / two / four
// / seven experts that every token names first or last 6.4 / 6.5 / 6.7 / 7.1 (6.6 / 8.1 / 11.2 / 16.0; 7.8 each); 16384
// tokens of one pair, all the same, 12.3 (11.2): top-1 is not looked at, which would cost it 2 %.
//
// Up to 512 tokens and 4096 pairs there are at most 8 workgroups, however many ranks.
//
// The workgroups' results fit together only if all of them saw one mask, see k_layout_small.  An instance of one
// context keeps its mask still.  A launch for an instance of several, or one captured before there were,
// learns it from the word behind the membership version; its workgroups use the mask that the first one read
// (agree_on), for a barrier and a round trip or two through memory more: T = 256 / 512 / 1024 / 2048
// 5.3 / 5.5 / 6.1 / 7.1 us.  (All of it done by the first workgroup took 8.6 / 11.1 / 19.3 / 29.9, and 65 for 2048 tokens of
// 8 ranks, and the loop over shares that it needed cost every launch 0.1 to 0.3 us.)
// ---------------------------------------------------------------------------
constexpr int kOnceThreads = 1024;
constexpr int kOnceMaxK = 10;  // compile-time top-k, a token to a lane, up to here
constexpr int kOncePairs = 16384, kShareTokens = 64, kPartPairs = 768;

// Element i of a small global array: a 32-bit offset from a scalar address, which takes no 64-bit
// arithmetic per lane.
template <class T>
__device__ __forceinline__ T& at(T* p, uint32_t i) {
  return *(T*)((char*)p + (uint32_t)(i * (uint32_t)sizeof(T)));
}

// What an expert's pairs need to know, one word per expert: the slot of its pairs from even tokens
// and << 12 that of those from odd ones.  Pairs without a row go to sinks behind the P slots, and
// are counted there: kDeadSinks for experts without a live replica, an expert to one of them, and kNoneSinks for what is
// no expert or a repeat, because counts of many lanes in one word come one after the other.
constexpr uint32_t kEntryMany = 1u << 24;  // more live ones to spread over: list start, count << 12
constexpr int kEntrySlots = 1 << 12;       // slots, sinks and counts stay below this
constexpr int kDeadSinks = 16, kNoneLanes = 8, kNoneSinks = kNoneLanes - 1 + kOnceMaxK;
constexpr int kSinks = kDeadSinks + kNoneSinks;

// Writes the entries of all experts and behind them those of no expert, and for experts with more than two live
// replicas to choose from the live ones to the front of the list.  The caller's next barrier makes both readable.
template <bool LARGE>
__device__ __forceinline__ void build_entries(const RouteTables& rt, uint32_t* entries, int E, int P,
                                              int policy, int nt) {
#pragma nounroll
  for (int e = threadIdx.x; e < E; e += nt) {  // (one pass unless LARGE)
    uint32_t even = P + (e & (kDeadSinks - 1)), odd = even, many = 0;
    const int o = rt.off[e], m = rt.off[e + 1] - o;
    const uint64_t two = (uint64_t)rt.alive[(o >> 5) + 1] << 32 | rt.alive[o >> 5];
    const uint32_t bits = (uint32_t)(two >> (o & 31)) & (uint32_t)((1ull << (m & 63)) - 1);
    const uint32_t rest = policy == EEP_FIRST_LIVE ? 0 : bits & (bits - 1);
    if (__builtin_expect(m > 32 || (rest & (rest - 1)) != 0, 0)) {
      int n = 0;
#pragma nounroll
      for (int q = o; q < o + m; ++q)
        if ((rt.alive[q >> 5] >> (q & 31)) & 1) rt.list[o + n++] = rt.list[q];
      if (n > 0) {
        many = kEntryMany;
        even = o;
        odd = policy == EEP_FIRST_LIVE ? 1 : n;
      }
    } else if (bits != 0) {
      even = odd = rt.list[o + __ffs(bits) - 1];
      if (rest != 0) odd = rt.list[o + __ffs(rest) - 1];
    }
    entries[e] = many | odd << 12 | even;
    if (!LARGE) break;
  }
  if (threadIdx.x < kNoneSinks) entries[E + threadIdx.x] = (P + kDeadSinks + threadIdx.x) * (1 + (1 << 12));
}

// A token's experts to their entries.  What is no expert goes to one of the kNoneSinks behind them, another one for each
// pair, so that it is no repeat either, and in kNoneLanes lanes; `none` is the lane's for the first pair.
template <uint32_t N>
__device__ __forceinline__ void entries_of(int (&e)[N], uint32_t none) {
#pragma unroll
  for (uint32_t j = 0; j < N; ++j) e[j] = min((uint32_t)e[j], none + j);
}

// Does a token name an expert twice?
template <uint32_t N>
__device__ __forceinline__ bool any_repeats(const int (&e)[N]) {
  uint32_t least = ~0u;
#pragma unroll
  for (uint32_t j = 1; j < N; ++j) {
#pragma unroll
    for (uint32_t i = 0; i < j; ++i) least = min(least, (uint32_t)(e[i] ^ e[j]));
  }
  return N > 1 && least == 0;
}

// The slots (or sinks) p[] of token t's pairs with the experts whose entries are e[].
template <uint32_t N>
__device__ __forceinline__ void map_token(const RouteTables& rt, const uint32_t* entries, int P, int (&e)[N],
                                          bool repeats, int t, int (&p)[N]) {
  uint32_t all = 0;
#pragma unroll
  for (uint32_t j = 0; j < N; ++j) p[j] = entries[e[j]];
#pragma unroll
  for (uint32_t j = 0; j < N; ++j) all |= p[j];
  if (__builtin_expect(__any(all >= kEntryMany), 0)) {
    // t % n by way of t / n in float, which is exact: (t + 0.5) / n is at least 0.5 / n away from an
    // integer, and t < 2^20
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) {
      const int lo = p[j] & (kEntrySlots - 1), hi = p[j] >> 12 & (kEntrySlots - 1);
      const int q = (int)(((float)t + 0.5f) * __builtin_amdgcn_rcpf((float)hi));
      int s = t & 1 ? hi : lo;
      if ((uint32_t)p[j] >= kEntryMany) s = rt.list[lo + t - q * hi];
      p[j] = s;
    }
  } else {
    const int shift = t & 1 ? 12 : 0;
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) p[j] = (uint32_t)p[j] >> shift & (kEntrySlots - 1);
  }
  if (__builtin_expect(__any(repeats), 0)) {  // (a router's choices never do)
#pragma unroll
    for (uint32_t j = 1; j < N; ++j) {
      asm volatile("" : "+v"(e[j]));  // (or the comparisons would be kept from above)
#pragma unroll
      for (uint32_t i = 0; i < j; ++i) p[j] = e[i] == e[j] ? P + kDeadSinks : p[j];
    }
  }
}

// Adds the lanes to counts[c], those of up to three different c (an expert's replicas) together, one lane for all: one
// word of LDS is otherwise added to by one lane after the other.
__device__ __forceinline__ void count_together(int32_t* counts, int c) {
  const int lane = threadIdx.x & 63;
  bool to_do = true;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (to_do) {
      const bool same = c == __builtin_amdgcn_readfirstlane(c);
      const int all = __popcll(__ballot(same));
      if (lane == __builtin_amdgcn_readfirstlane(lane)) atomicAdd(&counts[c], all);
      to_do = !same;
    }
  }
  if (to_do) atomicAdd(&counts[c], 1);
}
__device__ __forceinline__ bool same_in_all_lanes(int v) { return __all(v == __builtin_amdgcn_readfirstlane(v)); }

// Adds a token's pairs, of experts e[] in slots p[], to the counts from `region` on.  TOGETHER: lanes that have an
// expert in common are added by one of them.
template <uint32_t K, bool TOGETHER>
__device__ __forceinline__ void count_pairs(int32_t* s_cnt, uint32_t region, const int (&e)[K], const int (&p)[K]) {
  const bool all = TOGETHER && same_in_all_lanes(e[0]) && same_in_all_lanes(e[K - 1]);
  if (all) {
#pragma unroll
    for (uint32_t j = 0; j < K; ++j) count_together(s_cnt, region + p[j]);
  } else {
#pragma unroll
    for (uint32_t j = 0; j < K; ++j) {
      if (TOGETHER && same_in_all_lanes(e[j]))
        count_together(s_cnt, region + p[j]);
      else
        atomicAdd(&s_cnt[region + p[j]], 1);
    }
  }
}
// Keeps the slots p[] of a share's token tl, and marks it in their bitmaps.
template <uint32_t K>
__device__ __forceinline__ void keep_pairs(uint32_t* s_bm, uint32_t stride, int32_t* s_slot, uint32_t tl,
                                           const int (&p)[K]) {
  uint32_t* bm = s_bm + (tl >> 5);
  int32_t* to = s_slot + tl * K;
  const uint32_t bit = 1u << (tl & 31);
#pragma unroll
  for (uint32_t j = 0; j < K; ++j) to[j] = p[j];
#pragma unroll
  for (uint32_t j = 0; j < K; ++j) atomicOr(&bm[__umul24(p[j], stride)], bit);
}

// Bits [lo, hi) of a bitmap, lo < hi.
__device__ __forceinline__ int bits_between(const uint32_t* bm, int lo, int hi) {
  const int w0 = lo >> 5, w1 = (hi - 1) >> 5;
  int c = -__popc(bm[w0] & ~(~0u << (lo & 31)));
#pragma nounroll
  for (int w = w0; w < w1; ++w) c += __popc(bm[w]);
  return c + __popc(bm[w1] & ~0u >> (31 - ((hi - 1) & 31)));
}

// Counts per slot: tokens ahead of the share, its own, those behind it, and of these the ones that belong
// to the share's source rank where that is several shares and this its first.
__host__ __device__ constexpr int regions(bool parts) { return parts ? 4 : 3; }
// Tokens of a share: `ranks` whole source ranks, or one of `subs` parts of one.
__host__ __device__ inline uint32_t share_tokens(uint32_t tokens_per_rank, uint32_t ranks, uint32_t subs) {
  return subs == 1 ? ranks * tokens_per_rank : (tokens_per_rank + subs - 1) / subs;
}
// Words that start at zero: counts and bitmaps, a whole number of 16 bytes.
__host__ __device__ inline uint32_t once_zeros(uint32_t P, uint32_t stride, bool parts) {
  return ((P + kSinks) * (regions(parts) + stride) + 3) / 4 * 4;
}
// What starts at zero, tables, entries, offsets, a share's slots.
inline size_t once_lds_bytes(int E, int P, int R, int tokens, int k, bool parts) {
  return sizeof(int32_t) * ((size_t)once_zeros(P, token_stride(tokens), parts) + route_table_ints(E, P, R) +
                            (E + kNoneSinks) + (P + kSinks + 1) + (size_t)tokens * k);
}

// One word of the mask that all workgroups of a launch use where it may change meanwhile: the one that the first
// workgroup read, which it passes on in *word together with a 1.  It waits for nobody, so every other workgroup's
// wait ends; the bound (some seconds) is for a device that stops in between.
constexpr int kAgreePolls = 1 << 22;
__device__ __forceinline__ uint32_t agree_on(uint64_t* word, uint32_t mine) {
  uint64_t v = (uint64_t)1 << 32 | mine;
  if (blockIdx.x == 0) {
    __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): it is there before this workgroup counts itself
    return mine;
  }
  for (int polls = 0; polls < kAgreePolls; ++polls) {
    v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v >> 32 != 0) return (uint32_t)v;
    __builtin_amdgcn_s_sleep(1);
  }
  return mine;
}

// K: top-k.  PARTS: a share is a part of a source rank, one of `subs`, otherwise `ranks` whole ones.
// Four words hold the shape (T and tokens per rank; E and P; R and the source ranks of a share << 12;
// S, policy << 12, wavefronts << 13, shares in a rank << 18), so that it arrives in registers with the first pointers.
template <uint32_t K, bool LARGE, bool PARTS>
__global__ __launch_bounds__(kOnceThreads) void k_layout_once(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ l2p_off,
    const int32_t* __restrict__ l2p_list, const int32_t* __restrict__ active,
    const int32_t* __restrict__ mem_version, uint32_t T_rank, uint32_t E_P, uint32_t R_ranks,
    uint32_t S_policy_waves_subs, const int32_t* __restrict__ tbl_version, int32_t* __restrict__ slot_of,
    int32_t* __restrict__ row_of, int32_t* __restrict__ src_of, int32_t* __restrict__ cnt_src,
    int32_t* __restrict__ count, int32_t* __restrict__ offset, int32_t* __restrict__ rank_count,
    int32_t* __restrict__ rank_offset, int32_t* __restrict__ status,
    int32_t* __restrict__ step_epoch) {
  const uint32_t T = T_rank & 0xffff, tokens_per_rank = T_rank >> 16;
  const uint32_t E = E_P & 0xffff, P = E_P >> 16, P2 = P + kSinks;
  const uint32_t R = R_ranks & 0xfff, ranks = PARTS ? 1 : R_ranks >> 12;
  const uint32_t S = S_policy_waves_subs & 0xfff, policy = S_policy_waves_subs >> 12 & 1;
  const uint32_t waves = S_policy_waves_subs >> 13 & 31, nt = waves * 64;
  const uint32_t subs = PARTS ? S_policy_waves_subs >> 18 : 1;
  const uint32_t tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const auto load = [&](uint32_t t, int (&e)[K]) { __builtin_memcpy(e, &at(topk_idx, t * K), sizeof(e)); };
  // From the batch's last tokens, which the last threads take, to its first: the first threads have the tables to do.
  int t = (int)(T + tid) - (int)nt;
  int e[K];
  load(max(t, 0), e);
  RouteTableLoad<LARGE> tables = {l2p_off, l2p_list, active, (int)E, (int)R, (int)P, (int)nt};
  tables.fetch();
  // several contexts in the instance.  (A vector load: a scalar one would be waited for together with
  // every kernel argument.)
  const int several_v = vector_load(&mem_version[1]);

  extern __shared__ __align__(16) int32_t smem[];
  const uint32_t tokens = share_tokens(tokens_per_rank, ranks, subs), stride = token_stride(tokens);
  const uint32_t zeros = once_zeros(P, stride, PARTS);
  int32_t* const s_cnt = smem;                                      // [regions][P2] pairs per slot
  uint32_t* const s_bm = (uint32_t*)(s_cnt + regions(PARTS) * P2);  // [P2][stride] bitmap of the share's tokens per slot
  int32_t* const s_tab = smem + zeros;
  uint32_t* const s_entry = (uint32_t*)(s_tab + route_table_ints(E, P, R));  // [E+kNoneSinks]
  int32_t* const s_offset = (int32_t*)s_entry + E + kNoneSinks;     // [P2+1] exclusive scan of the totals
  int32_t* const s_slot = s_offset + P2 + 1;                        // [tokens*K] slots of the share's pairs
  __shared__ uint32_t s_agreed[2];
#pragma nounroll
  for (uint32_t i = tid * 4; i < zeros; i += nt * 4) *(int4*)(smem + i) = make_int4(0, 0, 0, 0);
  struct {
    uint64_t* words;
    bool several;
    uint32_t R;
    uint32_t* s_agreed;
    __device__ __forceinline__ uint64_t operator()(uint64_t mask) const {
      if (!several) return mask;
      const uint32_t tid = threadIdx.x;
      if (tid < (uint32_t)mask_words(R)) s_agreed[tid] = agree_on(words + tid, (uint32_t)(mask >> (tid * 32)));
      __syncthreads();
      return (uint64_t)(R > 32 ? s_agreed[1] : 0) << 32 | s_agreed[0];
    }
    __device__ __forceinline__ void operator()(uint32_t* mask) const {
      if (!several) return;
      const uint32_t tid = threadIdx.x;
      if (tid < (uint32_t)mask_words(R)) mask[tid] = agree_on(words + tid, mask[tid]);
      __syncthreads();
    }
  } agree = {(uint64_t*)(step_epoch + kAgreeMask), __builtin_amdgcn_readfirstlane(several_v) != 0, R, s_agreed};
  const RouteTables rt = tables.fill(s_tab, __builtin_amdgcn_rcpf((float)S), agree);
  int before = 0;  // workgroups that had the mask before this one
  if (agree.several && tid == 0)
    before = __hip_atomic_fetch_add(step_epoch + kAgreeCount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t share = blockIdx.x;
  // PARTS: the share's rank (share / subs, by way of float), and which of the rank's shares it is
  const uint32_t rank0 = !PARTS ? share * ranks : __builtin_amdgcn_readfirstlane(
      (uint32_t)(((float)share + 0.5f) * __builtin_amdgcn_rcpf((float)subs)));
  const uint32_t sub = PARTS ? share - rank0 * subs : 0, rank_end = (rank0 + 1) * tokens_per_rank;
  const uint32_t lo = PARTS ? min(rank0 * tokens_per_rank + sub * tokens, rank_end) : rank0 * tokens_per_rank;
  const uint32_t hi = min(lo + tokens, PARTS ? rank_end : T);
  __syncthreads();
  build_entries<LARGE>(rt, s_entry, E, P, policy, nt);
  // Tokens that are copies of one another (padding that is routed like any token, a router that has collapsed), or name
  // some experts all alike, are told by their first and last expert, those of a wavefront's first round for all: padding
  // is last.
  const bool copies = K > 1 && (same_in_all_lanes(e[0]) || same_in_all_lanes(e[K - 1]));
  const uint32_t none = E + (tid & (kNoneLanes - 1));
  if constexpr (K > 1) entries_of(e, none);
  bool repeats = any_repeats(e);
  __syncthreads();
  const auto count_tokens = [&](auto together) {
#pragma nounroll
    while (t >= 0) {
      const uint32_t now = t;
      t -= nt;
      int next[K];
      if (t >= 0) load(t, next);
      int p[K];
      if constexpr (K == 1) entries_of(e, none);  // (here it needs no branch)
      map_token<K>(rt, s_entry, P, e, repeats, now, p);
      // counted in the token's region, and if the token is the share's own, kept
      const bool own = now >= lo && now < hi;
      uint32_t region = own ? P2 : now < lo ? 0 : 2 * P2;
      asm volatile("" : "+v"(region));  // (or the tokens of a share would take a branch of their own)
      count_pairs<K, decltype(together)::value>(s_cnt, region, e, p);
      if (PARTS && sub == 0 && now >= hi && now < rank_end)
        count_pairs<K, decltype(together)::value>(s_cnt, 3 * P2, e, p);
      if (own) keep_pairs<K>(s_bm, stride, s_slot, now - lo, p);
      if (t >= 0) {
#pragma unroll
        for (uint32_t j = 0; j < K; ++j) e[j] = next[j];
        if constexpr (K > 1) {
          entries_of(e, none);
          repeats = any_repeats(e);
        }
      }
    }
  };
  if (__builtin_expect(copies, 0))
    count_tokens(std::true_type());
  else
    count_tokens(std::false_type());
  __syncthreads();
  // Between two barriers: the scan, and what does not need it.
  const uint32_t n = (hi - lo) * K, g0 = lo * K;
  const auto total = [=](uint32_t p) { return s_cnt[p] + s_cnt[P2 + p] + s_cnt[2 * P2 + p]; };
  scan_totals(total, s_offset, P2, wave, waves);
  const int version = share == 0 ? vector_load(tbl_version) + vector_load(mem_version) : 0;
  // pairs per (source rank, slot): the tokens of a source rank are a bit range
  if (sub == 0) {
    const uint32_t mine = min(R - rank0, ranks);
#pragma nounroll
    for (uint32_t p = tid; p < P; p += nt) {
      const uint32_t* bm = &s_bm[__umul24(p, stride)];
      uint32_t to = rank0 * P + p;
      if constexpr (PARTS) {
        at(cnt_src, to) = s_cnt[P2 + p] + s_cnt[3 * P2 + p];
      } else if (tokens <= 64) {
        uint64_t bits = bm[0];
        if (stride > 1) bits |= (uint64_t)bm[1] << 32;
        const uint64_t mask = ~0ull >> (64 - tokens_per_rank);
#pragma nounroll
        for (uint32_t b = 0; b < mine; ++b, to += P) {
          at(cnt_src, to) = __popcll(bits & mask);
          bits >>= tokens_per_rank;
        }
      } else {
#pragma nounroll
        for (uint32_t b = 0; b < mine; ++b, to += P)
          at(cnt_src, to) = bits_between(bm, b * tokens_per_rank, (b + 1) * tokens_per_rank);
      }
    }
  }
  uint32_t p = P;
  int row = -1;
  const auto place = [&](uint32_t i) {  // slot of the share's pair i, its row less the slot's offset
    p = s_slot[i];
    row = s_cnt[p] + rank_in_slot(&s_bm[p * stride], i / K);
  };
  if (tid < n) place(tid);
  __syncthreads();
  const int rows = s_offset[P];
#pragma nounroll
  for (uint32_t i = tid; i < n;) {
    const uint32_t g = g0 + i;
    int slot = -1;
    if (p < P) {
      slot = p;
      row += s_offset[p];
      at(src_of, row) = g;
    } else {
      row = -1;
    }
    at(slot_of, g) = slot;
    at(row_of, g) = row;
    if ((int)g >= rows) at(src_of, g) = -1;  // rows past the last routed pair
    i += nt;
    if (i < n) place(i);
  }
  if (share == 0)
    write_step_tables(nt, s_offset, s_offset[P + kDeadSinks] - rows, s_offset[P2] - s_offset[P + kDeadSinks], version,
                      count, offset, rank_count, rank_offset, status, step_epoch, R, S, P);
  if (agree.several && wave == 0 && __builtin_amdgcn_readfirstlane(before) == (int)gridDim.x - 1) {
    // every workgroup has the mask: zeros again for the next launch
#pragma nounroll
    for (uint32_t i = tid; i < (uint32_t)mask_words(R); i += 64)
      __hip_atomic_store(agree.words + i, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) __hip_atomic_store(step_epoch + kAgreeCount, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---------------------------------------------------------------------------
// Layout and dispatch in ONE launch, for captured steps of up to 2048 tokens: eep_dispatch makes the node that its layout
// left in the graph one of these (layout_pack_node).  Bound by latency: a launch of its own costs the dispatch 1.9 us and,
// behind it, a round trip for the row indices and the tokens.  Here every workgroup lays the whole batch out for itself,
// which all of them do at once, with its pieces of the tokens on their way meanwhile, and stores these as soon as it knows
// their rows; the layout's results are written by whoever has them at hand: a token's by the wavefront of its first
// piece, the pairs per source rank a rank to a workgroup.
//
// Measured, whole steps in graphs of 4 (32 ranks x 9 slots, top-8, bf16), in two launches and in one: 7168 channels, T = 32 / 96 /
// 256 / 320 / 640 / 2048 10.0 / 13.6 / 22.1 / 23.0 / 34.5 / 84.4 us and 8.8 / 12.3 / 19.1 / 20.3 / 31.6 / 82.9; 2048 channels, T = 32 / 256 / 512 /
// 1024 / 2048 8.95 / 12.0 / 15.4 / 24.4 / 32.1 and 7.9 / 10.4 / 13.1 / 18.3 / 31.1; fp8, 4096 channels, T = 128 / 448 / 960
// 17.2 / 26.9 / 41.3 and 15.1 / 25.9 / 39.2; top-2, 2048 channels, T = 160 / 992 9.05 / 12.2 and 7.6 / 10.6.  Part of it is
// that mid-sized receive rows are held in the L2s (rows.hpp) here, where all wavefronts store at once.
// ---------------------------------------------------------------------------
// The agreement on a mask, as in k_layout_once, for launches of hundreds of workgroups, up to 64 ranks: the first workgroup leaves the mask in eight places, one
// for the workgroups of each XCD (kAgreeGroups, kAgreeGroupInts), which are counted there too.  (In one place the loads and the
// counting come one after the other: a step with two contexts, 7168 channels, T = 32 / 256 / 640 10.6 / 21.1 / 38.9 us, 8.5 / 18.5 /
// 32.6 in this form; with one context 7.9 / 17.6 / 30.8.)
struct SpreadAgreedMask {
  int32_t* groups;  // [kAgreeGroups][kAgreeGroupInts]: workgroups counted, groups counted (in the first one), mask words
  bool several;
  uint32_t* s_agreed;
  __device__ __forceinline__ uint64_t* words(uint32_t group) const {
    return (uint64_t*)(groups + group * kAgreeGroupInts + 2);
  }
  __device__ __forceinline__ uint64_t operator()(uint64_t mask) const {
    if (!several) return mask;
    const uint32_t tid = threadIdx.x, word = tid & 1;
    const uint64_t mine = (uint64_t)1 << 32 | (uint32_t)(mask >> (word * 32));
    if (blockIdx.x == 0) {
      if (tid < 2 * kAgreeGroups) {
        __hip_atomic_store(words(tid >> 1) + word, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): it is there before this workgroup counts itself
      }
      return mask;
    }
    if (tid < 2) {
      uint64_t v = mine;  // (after the bound, as in agree_on)
      for (int polls = 0; polls < kAgreePolls; ++polls) {
        v = __hip_atomic_load(words(blockIdx.x & (kAgreeGroups - 1)) + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (v >> 32 != 0) break;
        __builtin_amdgcn_s_sleep(1);
      }
      s_agreed[tid] = (uint32_t)(v >> 32 != 0 ? v : mine);
    }
    __syncthreads();
    return (uint64_t)s_agreed[1] << 32 | s_agreed[0];
  }
  __device__ __forceinline__ void operator()(uint32_t*) const {}  // (more than 64 ranks: not here)
  // Thread 0, once the workgroup has the mask.  The last one of the last group: true.
  __device__ __forceinline__ bool arrive_last() const {
    const uint32_t group = blockIdx.x & (kAgreeGroups - 1);
    const int size = (int)(gridDim.x / kAgreeGroups);
    if (__hip_atomic_fetch_add(groups + group * kAgreeGroupInts, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != size - 1)
      return false;
    return __hip_atomic_fetch_add(groups + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == kAgreeGroups - 1;
  }
  // Zeros again for the next launch, by one wavefront of the workgroup that was the last.
  __device__ __forceinline__ void clear() const {
    const uint32_t lane = threadIdx.x & 63, group = lane >> 3, word = lane & 7;
    if (word < 6)
      __hip_atomic_store(groups + group * kAgreeGroupInts + word, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

// The piece of a wavefront of a launch that moves rows, see PackPieces: of token t, `vecs` vectors of a row of the
// payload or of the scales, the lane's from v on.
struct Piece {
  uint32_t t, part, v, vecs;
  bool any, scales;
};
// Pieces, counted token by token, go to the XCDs in turn as the workgroups do: workgroup b takes every eighth one from
// b mod 8 on, one to each of its first `waves` wavefronts.
__device__ __forceinline__ uint32_t piece_token(uint32_t wave, uint32_t waves, uint32_t parts, uint32_t magic) {
  return token_of((((blockIdx.x >> 3) * waves + wave) << 3) + (blockIdx.x & 7), parts, magic);
}
template <uint32_t U>
__device__ __forceinline__ Piece piece_of(uint32_t wave, uint32_t waves, uint32_t T, uint32_t parts, uint32_t magic,
                                          uint32_t row_vecs, uint32_t scale_vecs) {
  const uint32_t m = (((blockIdx.x >> 3) * waves + wave) << 3) + (blockIdx.x & 7), lane = threadIdx.x & 63;
  Piece p;
  p.t = token_of(m, parts, magic);
  p.part = m - p.t * parts;
  p.any = wave < waves && p.t < T;
  p.scales = scale_vecs > 0 && p.part == parts - 1;
  p.v = p.scales ? lane : p.part * (64 * U) + lane;
  p.vecs = p.scales ? scale_vecs : row_vecs;
  return p;
}
template <uint32_t U>
__device__ __forceinline__ void load_piece(const Piece& pc, const u32x4* x, const u32x4* x_scale, u32x4 (&d)[U]) {
  if (!pc.any) return;
  const u32x4* src = (pc.scales ? x_scale : x) + (int64_t)pc.t * pc.vecs;
#pragma unroll
  for (uint32_t u = 0; u < U; ++u) d[u] = __builtin_nontemporal_load(&src[min(pc.v + u * 64, pc.vecs - 1)]);
}
// Stores the piece to the token's K rows, lane j's `row` for pair j (-1: none).
template <uint32_t K, uint32_t U>
__device__ __forceinline__ void store_piece(const Piece& pc, int row, const u32x4 (&d)[U], u32x4* recv,
                                            u32x4* recv_scale, bool held) {
  u32x4* to = pc.scales ? recv_scale : recv;
  int r[K];
#pragma unroll
  for (uint32_t j = 0; j < K; ++j) r[j] = __builtin_amdgcn_readlane(row, j);
#pragma unroll
  for (uint32_t u = 0; u < U; ++u) asm volatile("" ::"v"(d[u]));
  const auto stores = [&](auto h) {
#pragma unroll
    for (uint32_t j = 0; j < K; ++j) {
      if (r[j] < 0) continue;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
        if (pc.v + u * 64 < pc.vecs)
          store_row_at<decltype(h)::value>(to, (int64_t)r[j] * (pc.vecs * 16), (pc.v + u * 64) * 16, d[u]);
    }
  };
  if (held)
    stores(std::true_type());
  else
    stores(std::false_type());
}

// Few pairs, at most one to each of the NT threads, built like k_layout_small.  T_waves: T, and << 16 the wavefronts with a piece, and << 31 `held`.
template <int K, int NT>
__global__ __launch_bounds__(NT) void k_layout_pack_small(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ l2p_off,
    const int32_t* __restrict__ l2p_list, const int32_t* __restrict__ active,
    const int32_t* __restrict__ mem_version, uint32_t T_waves, int E, int P, int R,
    const u32x4* __restrict__ x, uint32_t row_vecs, uint32_t parts, uint32_t magic,
    const u32x4* __restrict__ x_scale, uint32_t scale_vecs, float inv_S, int policy, int tokens_per_rank, int S,
    u32x4* __restrict__ recv, u32x4* __restrict__ recv_scale, const int32_t* __restrict__ tbl_version,
    int32_t* __restrict__ slot_of, int32_t* __restrict__ row_of, int32_t* __restrict__ src_of,
    int32_t* __restrict__ count, int32_t* __restrict__ offset, int32_t* __restrict__ rank_count,
    int32_t* __restrict__ rank_offset, int32_t* __restrict__ cnt_src,
    int32_t* __restrict__ status, int32_t* __restrict__ step_epoch) {
  const int T = T_waves & 0xffff, waves = T_waves >> 16 & 31;
  const bool held = T_waves >> 31 != 0;
  const int npairs = T * K;
  const int stride = token_stride(T);
  extern __shared__ int32_t smem[];
  int32_t* s_count = smem;                        // [P] pairs per slot
  uint32_t* s_bm = (uint32_t*)(s_count + P);      // [P][stride] token bitmap per slot
  int32_t* s_offset = (int32_t*)(s_bm + P * stride);  // [P+1] exclusive scan of s_count
  int32_t* s_slot = s_offset + P + 1;             // [T*K] slots of the pairs
  int32_t* s_tab = s_slot + npairs;
  __shared__ int32_t s_drop[2];
  __shared__ uint32_t s_agreed[2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // every global read of this kernel is issued here, none depends on another
  int my_e[1], slot[1];
  my_e[0] = tid < npairs ? topk_idx[tid] : -1;
  const int version = blockIdx.x == 0 && tid == 0 ? *tbl_version + *mem_version : 0;
  const int several_v = vector_load(&mem_version[1]);  // several contexts in the instance
  RouteTableLoad<false> tables = {l2p_off, l2p_list, active, E, R, P, NT};
  tables.fetch();
  const Piece pc = piece_of<1>(wave, waves, T, parts, magic, row_vecs, scale_vecs);
  u32x4 d[1];
  load_piece(pc, x, x_scale, d);
#pragma nounroll
  for (int i = tid; i < P * (stride + 1); i += NT) s_count[i] = 0;  // and s_bm
  if (tid < 2) s_drop[tid] = 0;
  const SpreadAgreedMask agree = {step_epoch + kAgreeGroupsAt, __builtin_amdgcn_readfirstlane(several_v) != 0, s_agreed};
  const RouteTables rt = tables.fill(s_tab, inv_S, agree);
  bool last = false;  // of the workgroups to have the mask (thread 0)
  if (agree.several && tid == 0) last = agree.arrive_last();
  __syncthreads();
  map_pairs<K, 1, NT>(rt, my_e, s_slot, slot, s_bm, stride, s_count, s_drop, npairs, K, E, 0, policy, 0, 0, slot_of);
  if (tid < npairs) s_slot[tid] = slot[0];
  __syncthreads();
  scan_totals([=](int p) { return s_count[p]; }, s_offset, P, wave, NT / 64);
  __syncthreads();

  const int N = s_offset[P];
  if (pc.any) {
    const int i = pc.t * K + (lane < K ? lane : K - 1);
    const int p = s_slot[i];
    const int row = p >= 0 ? s_offset[p] + rank_in_slot(&s_bm[p * stride], pc.t) : -1;
    store_piece<K>(pc, row, d, recv, recv_scale, held);
    if (pc.part == 0 && lane < K) {
      slot_of[i] = p;
      row_of[i] = row;
      if (p >= 0) src_of[row] = i;
      if (i >= N) src_of[i] = -1;  // rows past the last routed pair
    }
  }
  // pairs per (source rank, slot): the tokens of a source rank are a bit range
  for (int b = wave * gridDim.x + blockIdx.x; b < R; b += gridDim.x * (NT / 64)) {
    const int lo = b * tokens_per_rank, hi = lo + tokens_per_rank;
    int32_t* cnt = cnt_src + (int64_t)b * P;
    if (P <= 64)
      store_src_counts<1>(s_bm, stride, 0, P, lo, hi, cnt);
    else
      for (int p0 = 0; p0 < P; p0 += 320) store_src_counts<5>(s_bm, stride, p0, P, lo, hi, cnt);
  }
  if (blockIdx.x == 0)
    write_step_tables(NT, s_offset, s_drop[0], s_drop[1], version, count, offset, rank_count,
                      rank_offset, status, step_epoch, R, S, P);
  if (agree.several && wave == 0 && __builtin_amdgcn_readfirstlane(last)) agree.clear();
}

// More pairs, built like k_layout_once: a workgroup's share are the tokens that its pieces belong to, at most `window`,
// and for the pairs per source rank workgroup b counts rank b's beside it.  Words: T and tokens per
// rank; E and P; R and S << 12; `window`, policy << 12, wavefronts << 13, those with a piece << 18, `held` << 31.
template <uint32_t K, uint32_t U>
__global__ __launch_bounds__(kOnceThreads) void k_layout_pack_once(
    const int32_t* __restrict__ topk_idx, const int32_t* __restrict__ l2p_off,
    const int32_t* __restrict__ l2p_list, const int32_t* __restrict__ active,
    const int32_t* __restrict__ mem_version, uint32_t T_rank, uint32_t E_P, uint32_t R_S, uint32_t window_waves,
    const u32x4* __restrict__ x, uint32_t row_vecs, uint32_t parts, uint32_t magic,
    const u32x4* __restrict__ x_scale, uint32_t scale_vecs, u32x4* __restrict__ recv,
    u32x4* __restrict__ recv_scale, const int32_t* __restrict__ tbl_version, int32_t* __restrict__ slot_of,
    int32_t* __restrict__ row_of, int32_t* __restrict__ src_of, int32_t* __restrict__ cnt_src,
    int32_t* __restrict__ count, int32_t* __restrict__ offset, int32_t* __restrict__ rank_count,
    int32_t* __restrict__ rank_offset, int32_t* __restrict__ status,
    int32_t* __restrict__ step_epoch) {
  const uint32_t T = T_rank & 0xffff, tokens_per_rank = T_rank >> 16;
  const uint32_t E = E_P & 0xffff, P = E_P >> 16, P2 = P + kSinks;
  const uint32_t R = R_S & 0xfff, S = R_S >> 12;
  const uint32_t window = window_waves & 0xfff, policy = window_waves >> 12 & 1;
  const uint32_t waves = window_waves >> 13 & 31, nt = waves * 64, moving = window_waves >> 18 & 31;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const auto load = [&](uint32_t t, int (&e)[K]) { __builtin_memcpy(e, &at(topk_idx, t * K), sizeof(e)); };
  // From the batch's last tokens, which the last threads take, to its first: the first threads have the tables to do.
  int t = (int)(T + tid) - (int)nt;
  int e[K];
  load(max(t, 0), e);
  RouteTableLoad<false> tables = {l2p_off, l2p_list, active, (int)E, (int)R, (int)P, (int)nt};
  tables.fetch();
  const int several_v = vector_load(&mem_version[1]);  // several contexts in the instance
  const Piece pc = piece_of<U>(wave, moving, T, parts, magic, row_vecs, scale_vecs);
  u32x4 d[U];
  load_piece(pc, x, x_scale, d);

  extern __shared__ __align__(16) int32_t smem[];
  const uint32_t stride = token_stride(window);
  const uint32_t zeros = once_zeros(P, stride, true);
  int32_t* const s_cnt = smem;                                      // [regions][P2] pairs per slot
  uint32_t* const s_bm = (uint32_t*)(s_cnt + regions(true) * P2);   // [P2][stride] bitmap of the share's tokens per slot
  int32_t* const s_tab = smem + zeros;
  uint32_t* const s_entry = (uint32_t*)(s_tab + route_table_ints(E, P, R));  // [E+kNoneSinks]
  int32_t* const s_offset = (int32_t*)s_entry + E + kNoneSinks;     // [P2+1] exclusive scan of the totals
  int32_t* const s_slot = s_offset + P2 + 1;                        // [window*K] slots of the share's pairs
  __shared__ uint32_t s_agreed[2];
#pragma nounroll
  for (uint32_t i = tid * 4; i < zeros; i += nt * 4) *(int4*)(smem + i) = make_int4(0, 0, 0, 0);
  const SpreadAgreedMask agree = {step_epoch + kAgreeGroupsAt, __builtin_amdgcn_readfirstlane(several_v) != 0, s_agreed};
  const RouteTables rt = tables.fill(s_tab, __builtin_amdgcn_rcpf((float)S), agree);
  bool last = false;  // of the workgroups to have the mask (thread 0)
  if (agree.several && tid == 0) last = agree.arrive_last();
  const uint32_t lo = min(piece_token(0, moving, parts, magic), T);
  const uint32_t hi = min(piece_token(moving - 1, moving, parts, magic) + 1, T);
  const uint32_t rank_lo = blockIdx.x * tokens_per_rank, rank_hi = rank_lo + tokens_per_rank;  // (beyond T: none)
  __syncthreads();
  build_entries<false>(rt, s_entry, E, P, policy, nt);
  const bool copies = K > 1 && (same_in_all_lanes(e[0]) || same_in_all_lanes(e[K - 1]));  // see k_layout_once
  const uint32_t none = E + (tid & (kNoneLanes - 1));
  if constexpr (K > 1) entries_of(e, none);
  bool repeats = any_repeats(e);
  __syncthreads();
  const auto count_tokens = [&](auto together) {
#pragma nounroll
    while (t >= 0) {
      const uint32_t now = t;
      t -= nt;
      int next[K];
      if (t >= 0) load(t, next);
      int p[K];
      if constexpr (K == 1) entries_of(e, none);  // (here it needs no branch)
      map_token<K>(rt, s_entry, P, e, repeats, now, p);
      const bool own = now >= lo && now < hi;
      uint32_t region = own ? P2 : now < lo ? 0 : 2 * P2;
      asm volatile("" : "+v"(region));  // (or the tokens of a share would take a branch of their own)
      count_pairs<K, decltype(together)::value>(s_cnt, region, e, p);
      if (now >= rank_lo && now < rank_hi) count_pairs<K, decltype(together)::value>(s_cnt, 3 * P2, e, p);
      if (own) keep_pairs<K>(s_bm, stride, s_slot, now - lo, p);
      if (t >= 0) {
#pragma unroll
        for (uint32_t j = 0; j < K; ++j) e[j] = next[j];
        if constexpr (K > 1) {
          entries_of(e, none);
          repeats = any_repeats(e);
        }
      }
    }
  };
  if (__builtin_expect(copies, 0))
    count_tokens(std::true_type());
  else
    count_tokens(std::false_type());
  __syncthreads();
  // Between two barriers: the scan, and what does not need it.
  const auto total = [=](uint32_t p) { return s_cnt[p] + s_cnt[P2 + p] + s_cnt[2 * P2 + p]; };
  scan_totals(total, s_offset, P2, wave, waves);
  const int version = blockIdx.x == 0 ? vector_load(tbl_version) + vector_load(mem_version) : 0;
  const uint32_t j = lane < K ? lane : K - 1;
  uint32_t p = P;
  int row = -1;
  if (pc.any) {  // slot of the token's pair j, its row less the slot's offset
    const uint32_t tl = pc.t - lo;
    p = s_slot[tl * K + j];
    row = s_cnt[p] + rank_in_slot(&s_bm[p * stride], tl);
  }
  __syncthreads();
  const int rows = s_offset[P];
  if (pc.any) {
    row = p < P ? row + s_offset[p] : -1;
    store_piece<K>(pc, row, d, recv, recv_scale, window_waves >> 31 != 0);
    if (pc.part == 0 && lane < K) {
      const uint32_t g = pc.t * K + j;
      at(slot_of, g) = p < P ? (int)p : -1;
      at(row_of, g) = row;
      if (p < P) at(src_of, row) = g;
      if ((int)g >= rows) at(src_of, g) = -1;  // rows past the last routed pair
    }
  }
  if (blockIdx.x < R) {
#pragma nounroll
    for (uint32_t q = tid; q < P; q += nt) at(cnt_src, blockIdx.x * P + q) = s_cnt[3 * P2 + q];
  }
  if (blockIdx.x == 0)
    write_step_tables(nt, s_offset, s_offset[P + kDeadSinks] - rows, s_offset[P2] - s_offset[P + kDeadSinks], version,
                      count, offset, rank_count, rank_offset, status, step_epoch, R, S, P);
  if (agree.several && wave == 0 && __builtin_amdgcn_readfirstlane(last)) agree.clear();
}

// What a share holds: source ranks, or a part of one.
struct ShareSize {
  int ranks, subs;
  int tokens(int tokens_per_rank) const { return (int)share_tokens(tokens_per_rank, ranks, subs); }
  int count(int R) const { return subs > 1 ? R * subs : (R + ranks - 1) / ranks; }
};
// For at most `shares` of them, or (0) of about kShareTokens tokens.
static ShareSize share_size(int E, int P, int R, int tokens_per_rank, int k, int shares) {
  ShareSize s = {shares > 0 ? (R + shares - 1) / shares : kShareTokens / tokens_per_rank,
                 shares > 0 ? shares / R : (tokens_per_rank + kShareTokens / 2) / kShareTokens};
  if (s.ranks < 1) s.ranks = 1;
  if (s.subs < 1 || tokens_per_rank * k < kPartPairs || large_tables(E, P, R, kOnceThreads)) s.subs = 1;
  return s;
}

// ---------------------------------------------------------------------------
// Many tiles (> 64, the prefill regime): three launches.
//   k_tile_prefix  one workgroup per 64 slots (lane = slot, coalesced rows of the
//                  [tiles][P] count matrix); its 16 wavefronts split the tiles,
//                  each sums its share (one round of loads when the share is
//                  <= 32 tiles), the shares are combined through LDS, and every
//                  wavefront writes pre_tile[tile][slot] = pairs of the slot in
//                  earlier tiles, plus the slot totals.
//   k_position     a wide grid; every workgroup scans the P slot totals in LDS
//                  (cheap, and it saves a launch), then row = slot offset +
//                  earlier-tile pairs + rank in tile.  Workgroup 0 publishes the
//                  per-step tables.
// ---------------------------------------------------------------------------
constexpr int kPrefixThreads = 1024;
constexpr int kPrefixWaves = kPrefixThreads / 64;

__global__ __launch_bounds__(kPrefixThreads) void k_tile_prefix(
    const int32_t* __restrict__ cnt_tile, int32_t* __restrict__ pre_tile,
    int32_t* __restrict__ count, int num_tiles, int tiles_per_wave, int P) {
  __shared__ int32_t s_part[kPrefixWaves][64];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  const int b_lo = wave * tiles_per_wave;
  int b_hi = b_lo + tiles_per_wave;
  if (b_hi > num_tiles) b_hi = num_tiles;
  const bool single = tiles_per_wave <= kTileBatch;  // the share fits one batch: keep it in registers
  int v[kTileBatch];
  int part = 0;
  if (p < P) {
    for (int tb = b_lo; tb < b_hi; tb += kTileBatch) {
#pragma unroll
      for (int u = 0; u < kTileBatch; ++u)
        v[u] = tb + u < b_hi ? cnt_tile[(int64_t)(tb + u) * P + p] : 0;
#pragma unroll
      for (int u = 0; u < kTileBatch; ++u) part += v[u];
    }
  }
  s_part[wave][lane] = part;
  __syncthreads();
  if (p >= P) return;
  int run = 0;
  for (int w = 0; w < wave; ++w) run += s_part[w][lane];
  if (wave == 0) {
    int total = 0;
    for (int w = 0; w < kPrefixWaves; ++w) total += s_part[w][lane];
    count[p] = total;
  }
  for (int tb = b_lo; tb < b_hi; tb += kTileBatch) {
    if (!single) {
#pragma unroll
      for (int u = 0; u < kTileBatch; ++u)
        v[u] = tb + u < b_hi ? cnt_tile[(int64_t)(tb + u) * P + p] : 0;
    }
#pragma unroll
    for (int u = 0; u < kTileBatch; ++u) {
      if (tb + u < b_hi) pre_tile[(int64_t)(tb + u) * P + p] = run;
      run += v[u];
    }
  }
}

template <int KC>
__global__ __launch_bounds__(kPosThreads) void k_position(
    const int32_t* __restrict__ slot_of, const int32_t* __restrict__ pre_tile,
    const int32_t* __restrict__ count_in, const int32_t* __restrict__ blk_unc,
    const int32_t* __restrict__ blk_msk, const int32_t* __restrict__ tbl_version,
    const int32_t* __restrict__ mem_version, int32_t* __restrict__ row_of,
    int32_t* __restrict__ src_of, int32_t* __restrict__ cnt_src,
    int32_t* __restrict__ offset, int32_t* __restrict__ rank_count,
    int32_t* __restrict__ rank_offset, int32_t* __restrict__ status,
    int32_t* __restrict__ step_epoch, int k_rt, int tokens_per_rank, int tiles_per_rank,
    int tile_tokens, int num_tiles, int total_pairs, int R, int S, int P) {
  const int k = KC > 0 ? KC : k_rt;
  extern __shared__ int32_t smem[];
  int32_t* s_count = smem;           // [P]
  int32_t* s_offset = s_count + P;   // [P+1]
  __shared__ int32_t s_drop[2];
  const int tid = threadIdx.x;
  const int g = blockIdx.x * kPosThreads + tid;

  // this thread's pair, fetched together with the slot totals
  int p = -1, rank_in_tile = 0;
  if (g < total_pairs) {
    p = slot_of[g];
    rank_in_tile = row_of[g];
  }
  for (int q = tid; q < P; q += kPosThreads) s_count[q] = count_in[q];
  int du = 0, dm = 0, version = 0;
  if (blockIdx.x == 0) {
    for (int b = tid; b < num_tiles; b += kPosThreads) {
      du += blk_unc[b];
      dm += blk_msk[b];
    }
    if (tid == 0) version = *tbl_version + *mem_version;
  }
  if (tid < 2) s_drop[tid] = 0;
  __syncthreads();
  if (du) atomicAdd(&s_drop[0], du);
  if (dm) atomicAdd(&s_drop[1], dm);
  if (tid < 64) wave_exclusive_scan([=](int p) { return s_count[p]; }, s_offset, P);
  __syncthreads();

  // pairs per (source rank, slot): difference of the tile prefixes at the source
  // rank's first tile and at the next source rank's first tile
  for (int i = g; i < R * P; i += gridDim.x * kPosThreads) {
    int bs = i / P;
    int q = i - bs * P;
    int first = bs * tiles_per_rank, next = first + tiles_per_rank;
    int lo_v = pre_tile[(int64_t)first * P + q];
    int hi_v = next < num_tiles ? pre_tile[(int64_t)next * P + q] : s_count[q];
    cnt_src[i] = hi_v - lo_v;
  }
  if (g < total_pairs) {
    const int t = g / k;
    const int src_rank = t / tokens_per_rank;
    const int tile = src_rank * tiles_per_rank + (t - src_rank * tokens_per_rank) / tile_tokens;
    const int N = s_offset[P];
    int row = -1;
    if (p >= 0) {
      row = s_offset[p] + pre_tile[(int64_t)tile * P + p] + rank_in_tile;
      src_of[row] = g;
    }
    row_of[g] = row;
    if (g >= N) src_of[g] = -1;  // rows past the last routed pair
  }
  if (blockIdx.x == 0)
    write_step_tables(kPosThreads, s_offset, s_drop[0], s_drop[1], version, nullptr,
                                   offset, rank_count, rank_offset, status, step_epoch, R, S, P);
}

// T == 0: nothing is routed; publish empty tables.
__global__ __launch_bounds__(256) void k_empty_step(
    const int32_t* __restrict__ tbl_version, const int32_t* __restrict__ mem_version,
    int32_t* __restrict__ count, int32_t* __restrict__ offset, int32_t* __restrict__ rank_count,
    int32_t* __restrict__ rank_offset, int32_t* __restrict__ cnt_src,
    int32_t* __restrict__ status, int32_t* __restrict__ step_epoch, int R, int P) {
  for (int p = threadIdx.x; p <= P; p += 256) {
    offset[p] = 0;
    if (p < P) count[p] = 0;
  }
  for (int r = threadIdx.x; r <= R; r += 256) {
    rank_offset[r] = 0;
    if (r < R) rank_count[r] = 0;
  }
  for (int i = threadIdx.x; i < R * P; i += 256) cnt_src[i] = 0;
  if (threadIdx.x == 0) {
    status[0] = status[1] = status[2] = 0;
    status[3] = *tbl_version + *mem_version;
    *step_epoch = *step_epoch + 1;
  }
}

// ---------------------------------------------------------------------------
// De-duplicated dispatch (a data-path variant): one row per (token, destination
// rank).  Two launches after the ordinary layout, built like it: per tile a
// token bitmap per RANK gives the tile's count and the stable rank of a token
// inside the tile; then every workgroup derives the rank offsets and the pairs
// of earlier tiles from the small [tiles][R] count matrix.
//   dd_row[t,j]  row of token t in rank r's part of the rank-major buffer
//   dd_dst[t,j]  the same for the pair that carries the row (lowest j on that
//                rank), -1 for the others: the row table the pack kernel reads
//   dd_expand[row] for every expert-major row, the rank-major row behind it
// ---------------------------------------------------------------------------
template <int KC>
__global__ __launch_bounds__(kMapThreads) void k_dedup_count(
    const int32_t* __restrict__ slot_of, int32_t* __restrict__ dd_row,
    int32_t* __restrict__ dd_dst, int32_t* __restrict__ dd_tile, int k_rt, int R, int S,
    int tokens_per_rank, int tiles_per_rank, int tile_tokens) {
  const int k = KC > 0 ? KC : k_rt;
  extern __shared__ int32_t smem[];
  uint32_t* s_bm = (uint32_t*)smem;                       // [R][kBitmapWords]
  int32_t* s_slot = smem + R * kBitmapWords;              // [tile_tokens*k]
  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  const TileRange tr = tile_range(b, tokens_per_rank, tiles_per_rank, tile_tokens);
  const int npairs = tr.ntok * k;
  const int64_t g0 = (int64_t)tr.t0 * k;
  for (int i = tid; i < npairs; i += kMapThreads) s_slot[i] = slot_of[g0 + i];
  for (int i = tid; i < R * kBitmapWords; i += kMapThreads) s_bm[i] = 0u;
  __syncthreads();
  for (int i = tid; i < npairs; i += kMapThreads) {
    const int p = s_slot[i];
    if (p >= 0) {
      const int tl = i / k;
      atomicOr(&s_bm[(p / S) * kBitmapWords + (tl >> 5)], 1u << (tl & 31));
    }
  }
  __syncthreads();
  for (int i = tid; i < npairs; i += kMapThreads) {
    const int p = s_slot[i];
    int rank = -1, lead = 0;
    if (p >= 0) {
      const int r = p / S;
      const int tl = i / k;
      const int j = i - tl * k;
      lead = 1;
      for (int jj = 0; jj < j; ++jj) {
        const int q = s_slot[tl * k + jj];
        if (q >= 0 && q / S == r) lead = 0;
      }
      const uint32_t* bm = &s_bm[r * kBitmapWords];
      const int w = tl >> 5;
      rank = __popc(bm[w] & ((1u << (tl & 31)) - 1u));
      for (int ww = 0; ww < w; ++ww) rank += __popc(bm[ww]);
    }
    dd_row[g0 + i] = rank;  // rank inside the tile; the position kernel turns it into the row
    dd_dst[g0 + i] = lead;
  }
  for (int r = tid; r < R; r += kMapThreads) {
    int c = 0;
#pragma unroll
    for (int w = 0; w < kBitmapWords; ++w) c += __popc(s_bm[r * kBitmapWords + w]);
    dd_tile[(int64_t)b * R + r] = c;
  }
}

template <int KC>
__global__ __launch_bounds__(kMapThreads) void k_dedup_position(
    const int32_t* __restrict__ slot_of, const int32_t* __restrict__ row_of,
    const int32_t* __restrict__ src_of, const int32_t* __restrict__ offset,
    const int32_t* __restrict__ status, const int32_t* __restrict__ dd_tile,
    int32_t* __restrict__ dd_row, int32_t* __restrict__ dd_dst, int32_t* __restrict__ dd_expand,
    int32_t* __restrict__ dd_count, int32_t* __restrict__ dd_offset,
    int32_t* __restrict__ dd_status, int k_rt, int R, int S, int num_tiles, int tokens_per_rank,
    int tiles_per_rank, int tile_tokens) {
  const int k = KC > 0 ? KC : k_rt;
  extern __shared__ int32_t smem[];
  int32_t* s_cnt = smem;           // [R]   tokens per rank, all tiles
  int32_t* s_off = s_cnt + R;      // [R+1] exclusive scan of s_cnt
  int32_t* s_pre = s_off + R + 1;  // [R]   tokens per rank in tiles before this one
  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  const TileRange tr = tile_range(b, tokens_per_rank, tiles_per_rank, tile_tokens);
  const int npairs = tr.ntok * k;
  const int64_t g0 = (int64_t)tr.t0 * k;
  const int N = status[0];
  for (int r = tid; r < R; r += kMapThreads) {
    int total = 0, before = 0;
    for (int tb = 0; tb < num_tiles; tb += kTileBatch) {
      int v[kTileBatch];
#pragma unroll
      for (int u = 0; u < kTileBatch; ++u)
        v[u] = tb + u < num_tiles ? dd_tile[(int64_t)(tb + u) * R + r] : 0;
#pragma unroll
      for (int u = 0; u < kTileBatch; ++u) {
        total += v[u];
        before += tb + u < b ? v[u] : 0;
      }
    }
    s_cnt[r] = total;
    s_pre[r] = before;
  }
  __syncthreads();
  if (tid < 64) wave_exclusive_scan([=](int r) { return s_cnt[r]; }, s_off, R);
  __syncthreads();
  for (int i = tid; i < npairs; i += kMapThreads) {
    const int p = slot_of[g0 + i];
    int row_d = -1, dst = -1;
    if (p >= 0) {
      const int r = p / S;
      row_d = s_off[r] + s_pre[r] + dd_row[g0 + i];
      if (dd_dst[g0 + i] != 0) dst = row_d;
      const int row = row_of[g0 + i];
      if (row >= 0) {
        dd_expand[row] = row_d;
      } else {
        // withdrawn by failure detection since the layout: the slot's row that still names the
        // pair as its source gets no row of this step's (what stands there is an earlier step's)
        for (int q = offset[p]; q < offset[p + 1]; ++q)
          if (src_of[q] == (int)g0 + i) dd_expand[q] = -1;
      }
    }
    dd_row[g0 + i] = row_d;
    dd_dst[g0 + i] = dst;
    if (g0 + i >= N) dd_expand[g0 + i] = -1;  // rows past the last routed pair
  }
  if (b == 0) {
    for (int r = tid; r <= R; r += kMapThreads) {
      dd_offset[r] = s_off[r];
      if (r < R) dd_count[r] = s_cnt[r];
    }
    if (tid == 0) dd_status[0] = s_off[R];
  }
}

// The same in one launch for up to 64 ranks and kOncePairs pairs, built like k_layout_once: a workgroup
// owns 64 tokens, a lane takes a token (its ranks so far are a 64-bit mask), and every workgroup counts
// all tokens' ranks, those of tokens ahead of its own, its own and those behind apart.  Bound by latency;
// a launch of its own costs about 2 us beside that, and the host 2.6.  Whole de-duplicated steps in a graph
// of 8, the one-launch form of the ordinary layout on both sides: 2048 tokens over 8 ranks, 7168 channels,
// 158.3 us in two launches, 153.5 in one; 512 tokens 52.8 and 49.0.
// Few ranks are few LDS words, added to by one lane after the other.  There (BALLOT) a wavefront counts its 64 tokens by a
// ballot for each rank, which costs as much for every rank whatever its tokens: layout alone in a graph of 40, by lane / by
// ballot, top-1, 16320 tokens, 1 / 2 / 3 / 4 / 8 ranks 16.3 / 10.3 / 9.5 / 8.8 / 5.9 and 8.1 / 8.9 / 9.7 / 10.6 / 14.1 us; top-2, 8160
// tokens 10.1 / 9.4 / 8.4 / 7.7 / 6.5 and 5.8 / 6.2 / 6.7 / 7.1 / 8.8; top-4, 512 tokens 3.0 / 3.0 / 2.9 / 2.9 / 2.8 and 2.65 / 2.7 / 2.7 /
// 2.75 / 2.9; top-8, 2048 tokens, 1 / 2 / 4 / 8 / 12 / 16 ranks 5.5 / 5.95 / 6.1 / 5.95 / 5.7 / 5.5 and 4.4 / 4.5 / 4.7 / 5.1 / 5.6 / 5.9, 1024
// tokens of 8 ranks 4.2 and 4.3.  (In two launches top-1, 16320 tokens of up to 3 ranks took 9.0 to 10.1.)
constexpr int kDedupShare = 64;
static bool dedup_by_ballot(int R, int k, int T) {
  return R <= 4 ? R <= k + 1 : R <= 8 && k >= 6 && T > 1024;
}

template <int KC, bool BALLOT>
__global__ __launch_bounds__(kOnceThreads) void k_dedup_once(
    const int32_t* __restrict__ slot_of, const int32_t* __restrict__ row_of,
    const int32_t* __restrict__ status, int T, int R, int nt, float inv_S,
    const int32_t* __restrict__ src_of, const int32_t* __restrict__ offset,
    int32_t* __restrict__ dd_row, int32_t* __restrict__ dd_dst, int32_t* __restrict__ dd_expand,
    int32_t* __restrict__ dd_count, int32_t* __restrict__ dd_offset, int32_t* __restrict__ dd_status) {
  __shared__ int32_t s_cnt[3][64];             // tokens per rank
  __shared__ uint64_t s_bm[64];                // bitmap of the share's tokens per rank
  __shared__ int32_t s_first[64];              // rows ahead of the share's in each rank's part
  __shared__ int32_t s_pair[kDedupShare * KC]; // slot << 1, and whether the pair carries the row; -1
  const int tid = threadIdx.x;
  const int lo = blockIdx.x * kDedupShare, hi = lo + kDedupShare < T ? lo + kDedupShare : T;
  const int n = (hi - lo) * KC, g0 = lo * KC;
  int p[KC];
  __builtin_memcpy(p, &at(slot_of, (tid < T ? tid : T - 1) * KC), sizeof(p));
  const int my_row = at(row_of, g0 + (tid < n ? tid : 0));
  const int N = vector_load(status);
  if (tid < 64) {
    s_cnt[0][tid] = s_cnt[1][tid] = s_cnt[2][tid] = 0;
    s_bm[tid] = 0;
  }
  __syncthreads();
#pragma nounroll
  for (int t = tid; (BALLOT ? t - (tid & 63) : t) < T;) {
    const bool own = t >= lo && t < hi;
    // (with BALLOT whole wavefronts stay, whose tokens lie in one share)
    const int t0 = BALLOT ? __builtin_amdgcn_readfirstlane(t) : t;
    int32_t* cnt = s_cnt[t0 >= lo && t0 < hi ? 1 : t0 < lo ? 0 : 2];
    uint64_t mask = 0;
#pragma unroll
    for (int j = 0; j < KC; ++j) {
      bool lead = false;
      if (p[j] >= 0 && (!BALLOT || t < T)) {
        const int r = rank_of_slot(p[j], inv_S);
        lead = ((mask >> r) & 1) == 0;
        mask |= 1ull << r;
        if (!BALLOT && lead) {
          atomicAdd(&cnt[r], 1);
          if (own) atomicOr((unsigned long long*)&s_bm[r], 1ull << (t - lo));
        }
      }
      if (own) s_pair[(t - lo) * KC + j] = p[j] < 0 ? -1 : p[j] << 1 | lead;
    }
    if constexpr (BALLOT) {
      // A wavefront's 64 tokens lie in one share, so a ballot is a rank's count, and in the own share its bitmap;
      // lane r keeps rank r's.
      uint64_t mine = 0;
#pragma nounroll
      for (int r = 0; r < R; ++r) {
        const uint64_t has = __ballot((mask >> r) & 1);
        if ((tid & 63) == r) mine = has;
      }
      if ((tid & 63) < R) {
        if (t0 >= lo && t0 < hi) s_bm[tid & 63] = mine;
        atomicAdd(&cnt[tid & 63], __popcll(mine));
      }
    }
    t += nt;
    if (t < T) __builtin_memcpy(p, &at(slot_of, t * KC), sizeof(p));
  }
  __syncthreads();
  if (tid < 64) {
    const int all = s_cnt[0][tid] + s_cnt[1][tid] + s_cnt[2][tid];
    const int upto = wave_inclusive_scan(all);
    s_first[tid] = upto - all + s_cnt[0][tid];
    if (blockIdx.x == 0) {
      if (tid < R) dd_count[tid] = all;
      if (tid < R) dd_offset[tid] = upto - all;
      if (tid == R - 1) {
        dd_offset[R] = upto;
        dd_status[0] = upto;
      }
    }
  }
  __syncthreads();
#pragma nounroll
  for (int i = tid; i < n; i += nt) {
    const int v = s_pair[i], g = g0 + i;
    int row_d = -1, dst = -1;
    if (v >= 0) {
      const int r = rank_of_slot(v >> 1, inv_S);
      row_d = s_first[r] + __popcll(s_bm[r] & ((1ull << (i / KC)) - 1));
      if (v & 1) dst = row_d;
      const int row = i == tid ? my_row : at(row_of, g);
      if (row >= 0) {
        at(dd_expand, row) = row_d;
      } else {
        // withdrawn by failure detection since the layout, see k_dedup_position
        for (int q = offset[v >> 1]; q < offset[(v >> 1) + 1]; ++q)
          if (src_of[q] == g) dd_expand[q] = -1;
      }
    }
    at(dd_row, g) = row_d;
    at(dd_dst, g) = dst;
    if (g >= N) at(dd_expand, g) = -1;  // rows past the last routed pair
  }
}

hipError_t launch_dedup_layout(eep_ctx* c, int T, hipStream_t st) {
  Tiling g = make_tiling(T, c->R);
  if (g.num_tiles == 0) {
    hipError_t e = launch_fill(c->dd_count, 0, c->R, st);
    if (e == hipSuccess) e = launch_fill(c->dd_offset, 0, c->R + 1, st);
    if (e == hipSuccess) e = launch_fill(c->dd_status, 0, 1, st);
    return e;
  }
  if (c->R <= 64 && c->k <= kOnceMaxK && (int64_t)T * c->k <= kOncePairs) {
#define EEP_DEDUP(B) {k_dedup_once<1, B>, k_dedup_once<2, B>, k_dedup_once<3, B>, k_dedup_once<4, B>, k_dedup_once<5, B>, \
                      k_dedup_once<6, B>, k_dedup_once<7, B>, k_dedup_once<8, B>, k_dedup_once<9, B>, k_dedup_once<10, B>}
    static const decltype(&k_dedup_once<1, false>) of[2][kOnceMaxK] = {EEP_DEDUP(false), EEP_DEDUP(true)};
#undef EEP_DEDUP
    const bool ballot = dedup_by_ballot(c->R, c->k, T);
    const int nt = T > kOnceThreads ? kOnceThreads : kOnceThreads / 2;
    hipLaunchKernelGGL(of[ballot][c->k - 1], dim3((T + kDedupShare - 1) / kDedupShare), dim3(nt), 0, st, c->slot_of,
                       c->row_of, c->status, T, c->R, nt, 1.0f / (float)c->S, c->src_of, c->offset,
                       c->dd_row, c->dd_dst, c->dd_expand, c->dd_count, c->dd_offset, c->dd_status);
    return hipGetLastError();
  }
  const bool k8 = c->k == 8;
  {
    size_t lds = sizeof(int32_t) * ((size_t)c->R * kBitmapWords + (size_t)g.tile_tokens * c->k);
    auto kern = k8 ? k_dedup_count<8> : k_dedup_count<0>;
    hipLaunchKernelGGL(kern, dim3(g.num_tiles), dim3(kMapThreads), lds, st, c->slot_of, c->dd_row,
                       c->dd_dst, c->dd_tile, c->k, c->R, c->S, g.tokens_per_rank,
                       g.tiles_per_rank, g.tile_tokens);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  size_t lds = sizeof(int32_t) * ((size_t)3 * c->R + 1);
  auto kern = k8 ? k_dedup_position<8> : k_dedup_position<0>;
  hipLaunchKernelGGL(kern, dim3(g.num_tiles), dim3(kMapThreads), lds, st, c->slot_of, c->row_of,
                     c->src_of, c->offset, c->status, c->dd_tile, c->dd_row, c->dd_dst, c->dd_expand, c->dd_count,
                     c->dd_offset, c->dd_status, c->k, c->R, c->S, g.num_tiles, g.tokens_per_rank,
                     g.tiles_per_rank, g.tile_tokens);
  return hipGetLastError();
}

bool layout_shape_fits(int E, int P, int R, int k) {
  return map_lds_bytes(E, P, R, kTileTokens, k) <= kLayoutLdsLimit &&
         sizeof(int32_t) * ((size_t)3 * P + 1) <= kLayoutLdsLimit;
}

// The instantiation of a kernel family for top-k `k` and `pairs` pairs per workgroup of
// kMapThreads threads, at most 4 per thread: a compile-time k where the lanes of a token share a
// DPP row.
static_assert(kMaxPairsPerThread == 4, "widths of map_count_for");
template <int U, bool WIDE>
static auto map_count_for_k(int k) {
  return k == 8 ? k_map_count<8, U, WIDE> : k == 4 ? k_map_count<4, U, WIDE>
       : k == 2 ? k_map_count<2, U, WIDE> : k == 1 ? k_map_count<1, U, WIDE> : k_map_count<0, U, WIDE>;
}
template <bool WIDE>
static auto map_count_for(int k, int pairs) {
  return pairs <= kMapThreads ? map_count_for_k<1, WIDE>(k)
       : pairs <= 2 * kMapThreads ? map_count_for_k<2, WIDE>(k) : map_count_for_k<4, WIDE>(k);
}
template <bool LARGE>
static auto small_for(int k, int pairs) {
#define EEP_SMALL(U)                                                                              \
  (k == 8 ? k_layout_small<8, U, LARGE> : k == 4 ? k_layout_small<4, U, LARGE>                    \
   : k == 2 ? k_layout_small<2, U, LARGE> : k == 1 ? k_layout_small<1, U, LARGE> : k_layout_small<0, U, LARGE>)
  return pairs <= kMapThreads ? EEP_SMALL(1) : pairs <= 2 * kMapThreads ? EEP_SMALL(2) : EEP_SMALL(4);
#undef EEP_SMALL
}
template <bool LARGE, bool PARTS>
static auto once_for(int k) {
  static const decltype(&k_layout_once<1, LARGE, PARTS>) of[kOnceMaxK] = {
      k_layout_once<1, LARGE, PARTS>, k_layout_once<2, LARGE, PARTS>, k_layout_once<3, LARGE, PARTS>,
      k_layout_once<4, LARGE, PARTS>, k_layout_once<5, LARGE, PARTS>, k_layout_once<6, LARGE, PARTS>,
      k_layout_once<7, LARGE, PARTS>, k_layout_once<8, LARGE, PARTS>, k_layout_once<9, LARGE, PARTS>,
      k_layout_once<10, LARGE, PARTS>};
  return of[k - 1];
}

// Does an output array overlap the router indices (a caller that gives up its indices for the
// result)?  The workgroups of a one-launch form read all of them while others write already; one alone
// has read everything before it writes, and in the tiled form a workgroup reads its own pairs'
// before it writes these.
static bool writes_its_input(const LayoutIO& c, int T) {
  const int64_t pairs = (int64_t)T * c.k;
  const struct { const int32_t* p; int64_t n; } out[] = {
      {c.slot_of, pairs}, {c.row_of, pairs}, {c.src_of, pairs}, {c.count, c.P},
      {c.offset, c.P + 1}, {c.rank_count, c.R}, {c.rank_offset, c.R + 1},
      {c.cnt_src, (int64_t)c.R * c.P}, {c.status, 4}};
  const uintptr_t lo = (uintptr_t)c.topk_idx, hi = lo + pairs * sizeof(int32_t);
  for (const auto& o : out)
    if ((uintptr_t)o.p < hi && lo < (uintptr_t)(o.p + o.n)) return true;
  return false;
}

// Workgroups of a one-launch form for a small batch; 0: larger, or its tables do not fit.  `solo`: more
// than one could disagree (the mask may change while the kernel runs, or an output overlaps the input).
int layout_small_workgroups(int E, int P, int R, int T, int k, bool solo) {
  if (T < 1 || T > (solo ? kSoloTokens : kSmallTokens) ||
      T * k > (solo ? kSoloPairs : kSmallPairs) || small_lds_bytes(E, P, R, T, k) > kLayoutLdsLimit)
    return 0;
  return solo ? 1 : kSmallBlocks;
}

hipError_t launch_layout(const LayoutIO& c, int T, hipStream_t st, bool* one_launch) {
  Tiling g = make_tiling(T, c.R);
  const bool k8 = c.k == 8;
  if (one_launch != nullptr) *one_launch = true;
  if (g.num_tiles == 0) {
    hipLaunchKernelGGL(k_empty_step, dim3(1), dim3(256), 0, st, c.tbl_version, c.mem_version,
                       c.count, c.offset, c.rank_count, c.rank_offset, c.cnt_src, c.status,
                       c.step_epoch, c.R, c.P);
    return hipGetLastError();
  }
  if (g.num_tiles > max_blocks(kMapThreads)) return hipErrorInvalidValue;
  const float inv_S = 1.0f / (float)c.S;
  const bool overlaps = writes_its_input(c, T), solo = c.mask_may_change || overlaps;
  const int small = layout_small_workgroups(c.E, c.P, c.R, T, c.k, solo);
  // Several contexts: beyond the sizes for one workgroup, k_layout_once with its workgroups' agreement on a mask is
  // faster than tiles (32 ranks x 9 slots, a layout in a graph of 40; top-8, T = 416 / 512 / 1024 / 2048: 5.6 / 5.4 / 6.1 / 7.05 us,
  // in tiles 7.75 / 7.5 / 7.7 / 7.8; top-2, T = 512 / 4096 4.8 / 5.85 (7.4 / 7.7); all tokens alike, T = 2048 7.65 (7.6)).
  const bool agree = c.mask_may_change && c.can_agree && !overlaps && small == 0;
  const ShareSize share = share_size(c.E, c.P, c.R, g.tokens_per_rank, c.k,
                                     agree ? layout_small_workgroups(c.E, c.P, c.R, T, c.k, false) : small);
  const int tokens = share.tokens(g.tokens_per_rank);
  const bool has_k = c.k == 1 || c.k == 2 || c.k == 4 || c.k == 8;  // an instance of k_layout_small
  const bool few = small > 0 && has_k && T * c.k <= kFewPairs;
  if ((!solo || agree) && !few && c.k <= kOnceMaxK && (int64_t)T * c.k <= kOncePairs && c.P + kSinks <= kEntrySlots &&
      once_lds_bytes(c.E, c.P, c.R, tokens, c.k, share.subs > 1) <= kLayoutLdsLimit) {
    int nt = c.P > c.E ? c.P : c.E + 1;  // threads: for the tables, and for the tokens
    const int most = T > kOnceThreads ? kOnceThreads : kOnceThreads / 2;
    nt = nt < most ? most : nt < kOnceThreads ? (nt + 63) / 64 * 64 : kOnceThreads;
    auto kern = large_tables(c.E, c.P, c.R, nt) ? once_for<true, false>(c.k)
                : share.subs > 1 ? once_for<false, true>(c.k) : once_for<false, false>(c.k);
    hipLaunchKernelGGL(kern, dim3(share.count(c.R)), dim3(nt),
                       once_lds_bytes(c.E, c.P, c.R, tokens, c.k, share.subs > 1), st, c.topk_idx,
                       c.l2p_off, c.l2p_list, c.active, c.mem_version,
                       (uint32_t)T | (uint32_t)g.tokens_per_rank << 16, (uint32_t)c.E | (uint32_t)c.P << 16,
                       (uint32_t)c.R | (uint32_t)share.ranks << 12,
                       (uint32_t)c.S | (uint32_t)c.policy << 12 | (uint32_t)(nt / 64) << 13 |
                           (uint32_t)share.subs << 18,
                       c.tbl_version, c.slot_of, c.row_of,
                       c.src_of, c.cnt_src, c.count, c.offset, c.rank_count, c.rank_offset, c.status,
                       c.step_epoch);
    return hipGetLastError();
  }
  if (small > 0) {
    auto kern = large_tables(c.E, c.P, c.R, kMapThreads) ? small_for<true>(c.k, T * c.k) : small_for<false>(c.k, T * c.k);
    hipLaunchKernelGGL(kern, dim3(small), dim3(kMapThreads), small_lds_bytes(c.E, c.P, c.R, T, c.k),
                       st, c.topk_idx, c.l2p_off, c.l2p_list, c.active, c.mem_version,
                       (uint32_t)T | (uint32_t)c.k << 16 | (solo ? kSoloBit : 0u), c.E,
                       c.P, c.R, inv_S, c.tbl_version, c.policy, g.tokens_per_rank, c.S,
                       c.slot_of, c.row_of, c.src_of, c.count, c.offset, c.rank_count,
                       c.rank_offset, c.cnt_src, c.status, c.step_epoch);
    return hipGetLastError();
  }
  if (one_launch != nullptr) *one_launch = false;
  {
    size_t lds = sizeof(int32_t) * map_lds_ints(c.E, c.P, c.R, g.tile_tokens, c.k);
    auto kern = large_tables(c.E, c.P, c.R, kMapThreads) ? map_count_for<true>(c.k, g.tile_tokens * c.k) : map_count_for<false>(c.k, g.tile_tokens * c.k);
    hipLaunchKernelGGL(kern, dim3(g.num_tiles), dim3(kMapThreads), lds, st, c.topk_idx, c.l2p_off,
                       c.l2p_list, c.active, c.k, g.tokens_per_rank, g.tiles_per_rank,
                       g.tile_tokens, c.E, c.P, c.R, inv_S, c.policy, c.slot_of, c.row_of,
                       c.cnt_tile, c.blk_unc, c.blk_msk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const bool fused = g.num_tiles <= 64 && g.tile_tokens * c.k <= kFusedThreads * kFusedPairs;
  if (fused) {
    size_t lds = sizeof(int32_t) * ((size_t)3 * c.P + 1);
    auto kern = k8 ? k_scan_position<8> : k_scan_position<0>;
    hipLaunchKernelGGL(kern, dim3(g.num_tiles), dim3(kFusedThreads), lds, st, c.cnt_tile,
                       c.slot_of, c.row_of, c.P, g.num_tiles, c.k, g.tokens_per_rank,
                       g.tiles_per_rank, g.tile_tokens, c.blk_unc, c.blk_msk, c.tbl_version,
                       c.mem_version, c.R, c.S, c.src_of, c.count, c.offset, c.rank_count,
                       c.rank_offset, c.cnt_src, c.status, c.step_epoch);
    return hipGetLastError();
  }
  int tiles_per_wave = (g.num_tiles + kPrefixWaves - 1) / kPrefixWaves;
  hipLaunchKernelGGL(k_tile_prefix, dim3((c.P + 63) / 64), dim3(kPrefixThreads), 0, st, c.cnt_tile,
                     c.base_tile, c.count, g.num_tiles, tiles_per_wave, c.P);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int total_pairs = T * c.k;
  size_t lds_pos = sizeof(int32_t) * ((size_t)2 * c.P + 1);
  auto kern = k8 ? k_position<8> : k_position<0>;
  hipLaunchKernelGGL(kern, dim3((total_pairs + kPosThreads - 1) / kPosThreads), dim3(kPosThreads),
                     lds_pos, st, c.slot_of, c.base_tile, c.count, c.blk_unc, c.blk_msk,
                     c.tbl_version, c.mem_version, c.row_of, c.src_of, c.cnt_src, c.offset,
                     c.rank_count, c.rank_offset, c.status, c.step_epoch, c.k, g.tokens_per_rank,
                     g.tiles_per_rank, g.tile_tokens, g.num_tiles, total_pairs, c.R, c.S, c.P);
  return hipGetLastError();
}

static LayoutIO layout_io(eep_ctx* c, const int32_t* topk_idx) {
  LayoutIO io;
  io.R = c->R; io.S = c->S; io.P = c->P; io.E = c->E; io.k = c->k; io.policy = c->cfg.policy;
  io.topk_idx = topk_idx;
  io.mask_may_change = c->mem->members.size() > 1;
  io.can_agree = true;
  io.l2p_off = c->l2p_off; io.l2p_list = c->l2p_list; io.active = c->active;
  io.tbl_version = c->tbl_version; io.mem_version = c->mem->mem_version;
  io.slot_of = c->slot_of; io.row_of = c->row_of; io.src_of = c->src_of;
  io.count = c->count; io.offset = c->offset; io.rank_count = c->rank_count;
  io.rank_offset = c->rank_offset; io.cnt_src = c->cnt_src; io.status = c->status;
  io.cnt_tile = c->cnt_tile; io.base_tile = c->base_tile; io.blk_unc = c->blk_unc;
  io.blk_msk = c->blk_msk; io.step_epoch = c->step_epoch;
  return io;
}

hipError_t launch_layout(eep_ctx* c, const int32_t* topk_idx, int T, hipStream_t st, bool* one_launch) {
  return launch_layout(layout_io(c, topk_idx), T, st, one_launch);
}

// The widths of a piece, us a step in graphs of 4 with 1 / 2 / 4 / 7 KiB: top-8, 512 tokens of 10 KiB 23.25 / 24.4 / 24.4 / 23.8, 640 of
// 14 KiB 34.2 / 31.2 / 32.05 / 31.7, 768 of 8 KiB 23.0 / 23.9 / 27.0 / 30.0, 1024 of 7 KiB 28.6 / 27.7 / 27.7 / 27.3; top-4, 1024 of 14 KiB
// 29.6 / 29.6 / 28.2 / 28.1; top-2, 1536 of 8 KiB 19.3 / 16.6 / 17.4 / 18.7, 2048 of 4 KiB 17.3 / 14.9 / 15.8 / 15.9.  A top-k that is
// not here would take two launches, 1.14 times as long over 360 shapes of top-1 to 10.
template <uint32_t U>
static const void* layout_pack_once_for(int k) {
  static const decltype(&k_layout_pack_once<1, U>) of[kOnceMaxK] = {
      k_layout_pack_once<1, U>, k_layout_pack_once<2, U>, k_layout_pack_once<3, U>, k_layout_pack_once<4, U>,
      k_layout_pack_once<5, U>, k_layout_pack_once<6, U>, k_layout_pack_once<7, U>, k_layout_pack_once<8, U>,
      k_layout_pack_once<9, U>, k_layout_pack_once<10, U>};
  return (const void*)of[k - 1];
}

// How many pieces a workgroup takes.  More pieces than 8 wavefronts of every CU make further rounds of workgroups, which are
// resident together up to three (stay_resident), and in these all CUs are to get the same: 320 tokens of 7168 channels took
// 25.6 us a step with 16 wavefronts in 280 workgroups (35 for the 32 CUs of an XCD), 21.9 with 10 in 448, 21.7 with 6 in 752, 21.6 with 9 in
// 504.  One even round of more wavefronts is no better, though the batch is then laid out once on a CU: T = 160 / 192 / 224 / 256 / 288 (9 to 16
// wavefronts, 1024 threads) 16.15 / 17.3 / 18.6 / 19.3 / 21.8 us, two rounds of 512 threads 15.8 / 16.9 / 18.1 / 18.8 / 21.3, three 15.7 /
// 16.8 / 18.0 / 18.7 / 21.4; with a skewed router the same (T = 256 19.15 / 18.8 / 18.7).  Beyond three rounds (768 pieces to an XCD; 896 tokens of 7168 channels) two launches are as fast, and with three
// rounds of many pairs, all of which every workgroup lays out: two launches' time over that of one, 1088 channels, 288 slots,
// top-4 1536 / 2048 tokens 1.09 / 1.06, top-8 1.05 / 1.01; with a skewed router 1.03 / 0.975 and 0.98 / 0.935.
constexpr int kLayoutPackTokens = 2048, kXcdCus = 32, kPieceWaves = 8, kPieceRounds = 3, kThirdRoundPairs = 6144;

// Are `rounds` workgroups of nt threads resident on a CU together?  A round that has to wait for the one before lays the
// batch out again when that has ended: three rounds of top-10 (83 registers, 5 wavefronts to a SIMD), 1536 tokens of 1088
// channels 25.0 us a step, in two launches 22.1; of 576 slots (9 wavefronts, 3 of them on one SIMD) top-4 17.0 and 15.9; two rounds
// of both, 1024 tokens, 21.3 and 19.8.
static bool stay_resident(const void* kernel, int nt, int rounds) {
  hipFuncAttributes a;
  if (rounds <= 1) return true;
  if (hipFuncGetAttributes(&a, kernel) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  // wavefronts of a SIMD: 512 vector registers in eights, and the scalar ones are enough for 7
  const int waves = std::min(7, 512 / std::max(8, (a.numRegs + 7) / 8 * 8));
  return rounds * ((nt + 255) / 256) <= waves;
}

bool layout_pack_node(eep_ctx* ctx, const int32_t* topk_idx, PackPieces pk, int T, hipGraphNode_t node) {
  LayoutIO io = layout_io(ctx, topk_idx);
  const Tiling g = make_tiling(T, io.R);
  if (T < 1 || T > kLayoutPackTokens || io.k > kOnceMaxK || T * io.k > kOncePairs || io.P + kSinks > kEntrySlots ||
      writes_its_input(io, T))
    return false;
  const int pieces = (int)((T * (int64_t)pk.parts + 7) / 8);  // of an XCD
  if (pieces > kXcdCus * kPieceWaves * kPieceRounds) return false;
  // As k_layout_small up to the same size for top-4 and 8 (7168 channels, top-8, T = 32 / 96: 8.75 / 12.3 us, as k_layout_once
  // 9.0 / 12.6; for top-1 and 2 the latter is faster: T = 32 7.7 and 7.5).
  const bool few = (io.k == 4 || io.k == 8) && T * io.k <= kFewPairs && pk.vecs == 1 && pieces <= kXcdCus * 16 &&
                   !large_tables(io.E, io.P, io.R, kMapThreads) &&
                   small_lds_bytes(io.E, io.P, io.R, T, io.k) <= kLayoutLdsLimit;
  const int rounds = few ? 1 : (pieces + kXcdCus * kPieceWaves - 1) / (kXcdCus * kPieceWaves);
  const int waves = (pieces + kXcdCus * rounds - 1) / (kXcdCus * rounds);
  int grid = (pieces + waves - 1) / waves * 8;
  if (grid < io.R) grid = (io.R + 7) / 8 * 8;
  const uint32_t held = pk.held ? 1u << 31 : 0;
  uint32_t magic = part_magic((int)pk.parts, (int64_t)(grid + 8) * waves);
  if (few) {
    uint32_t T_waves = (uint32_t)T | (uint32_t)waves << 16 | held;
    int tokens_per_rank = g.tokens_per_rank;
    float inv_S = 1.0f / (float)io.S;
    void* args[] = {&io.topk_idx, &io.l2p_off, &io.l2p_list, &io.active, &io.mem_version, &T_waves, &io.E, &io.P, &io.R,
                    &pk.x, &pk.row_vecs, &pk.parts, &magic, &pk.x_scale, &pk.scale_vecs, &inv_S, &io.policy,
                    &tokens_per_rank, &io.S, &pk.recv, &pk.recv_scale, &io.tbl_version, &io.slot_of, &io.row_of,
                    &io.src_of, &io.count, &io.offset, &io.rank_count, &io.rank_offset, &io.cnt_src, &io.status,
                    &io.step_epoch};
    // (half the threads where there is a pair to each: T = 32 / 64 7.65 / 9.5 us a step, 7.85 / 9.75 with 16 wavefronts)
    const bool half = T * io.k <= kMapThreads / 2 && waves <= kMapThreads / 128 &&
                      !large_tables(io.E, io.P, io.R, kMapThreads / 2);
    return set_node(node,
                    half ? (io.k == 8 ? (const void*)k_layout_pack_small<8, kMapThreads / 2>
                                      : (const void*)k_layout_pack_small<4, kMapThreads / 2>)
                         : (io.k == 8 ? (const void*)k_layout_pack_small<8, kMapThreads>
                                      : (const void*)k_layout_pack_small<4, kMapThreads>),
                    grid, half ? kMapThreads / 2 : kMapThreads, small_lds_bytes(io.E, io.P, io.R, T, io.k), args);
  }
  int nt = kOnceThreads / 2;  // threads: for the tables too
  while (nt < kOnceThreads && large_tables(io.E, io.P, io.R, nt)) nt += 64;
  const int window = 8 * (waves - 1) / (int)pk.parts + 2;  // the most tokens that a workgroup's pieces belong to
  const size_t lds = once_lds_bytes(io.E, io.P, io.R, window, io.k, true);
  const void* const kernel = pk.vecs == 1   ? layout_pack_once_for<1>(io.k)
                             : pk.vecs == 2 ? layout_pack_once_for<2>(io.k)
                             : pk.vecs == 4 ? layout_pack_once_for<4>(io.k) : layout_pack_once_for<7>(io.k);
  if (lds > kLayoutLdsLimit || large_tables(io.E, io.P, io.R, nt) ||
      (rounds == kPieceRounds && T * io.k > kThirdRoundPairs) || !stay_resident(kernel, nt, rounds))
    return false;
  uint32_t T_rank = (uint32_t)T | (uint32_t)g.tokens_per_rank << 16, E_P = (uint32_t)io.E | (uint32_t)io.P << 16;
  uint32_t R_S = (uint32_t)io.R | (uint32_t)io.S << 12;
  uint32_t window_waves = (uint32_t)window | (uint32_t)io.policy << 12 | (uint32_t)(nt / 64) << 13 |
                          (uint32_t)waves << 18 | held;
  void* args[] = {&io.topk_idx, &io.l2p_off, &io.l2p_list, &io.active, &io.mem_version, &T_rank, &E_P, &R_S,
                  &window_waves, &pk.x, &pk.row_vecs, &pk.parts, &magic, &pk.x_scale, &pk.scale_vecs, &pk.recv,
                  &pk.recv_scale, &io.tbl_version, &io.slot_of, &io.row_of, &io.src_of, &io.cnt_src, &io.count,
                  &io.offset, &io.rank_count, &io.rank_offset, &io.status, &io.step_epoch};
  return set_node(node, kernel, grid, nt, lds, args);
}

}  // namespace eep

extern "C" int eep_host_layout_workgroups(int32_t R, int32_t S, int32_t E, int32_t k, int32_t T,
                                          int32_t several_contexts) {
  if (R < 1 || S < 1 || E < 1 || k < 1 || k > eep::kMaxTopk || T < 0 || T % R != 0 ||
      (int64_t)R * S > (1 << 20) || E > (1 << 20) || (int64_t)T * k > (int64_t)1 << 30)
    return EEP_ERR_INVALID_ARG;
  return eep::layout_small_workgroups(E, R * S, R, T, k, several_contexts != 0);
}
