// Weight movement for a planned repair (paper Sec. 3.5: local reuse, batched
// GPU-to-GPU relocation, reload from the DRAM backup; Sec. 5.1: the active mask
// is looked up when a transfer is issued).  One kernel moves the whole batch.
#include <string.h>

#include <algorithm>
#include <vector>

#include "eep_internal.hpp"

using namespace eep;

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMoveThreads = 256;
constexpr int kMoveVecs = 8;                                            // 16-byte vectors per thread per pass
constexpr int kMovePasses = 2;
constexpr int kChunkVecs = kMoveThreads * kMoveVecs * kMovePasses;      // 64 KiB per workgroup

// Copies chunk `chunk` of a move.  Source and destination both lie in `weights` for a peer copy, so no restrict.
__device__ __forceinline__ void copy_chunk(u32x4* weights, const u32x4* backup, int64_t slot_vecs, int chunk,
                                           int dst, int src, int expert, bool from_peer) {
  const u32x4* from = from_peer ? weights + (int64_t)src * slot_vecs : backup + (int64_t)expert * slot_vecs;
  u32x4* to = weights + (int64_t)dst * slot_vecs;
  const int64_t first = (int64_t)chunk * kChunkVecs + threadIdx.x;
  if ((int64_t)(chunk + 1) * kChunkVecs <= slot_vecs) {
    // full chunk: no per-vector guards, so all loads of a pass are in flight together
#pragma unroll
    for (int pass = 0; pass < kMovePasses; ++pass) {
      const int64_t base = first + (int64_t)pass * (kMoveThreads * kMoveVecs);
      u32x4 buf[kMoveVecs];
#pragma unroll
      for (int u = 0; u < kMoveVecs; ++u)
        buf[u] = __builtin_nontemporal_load(from + base + (int64_t)u * kMoveThreads);
#pragma unroll
      for (int u = 0; u < kMoveVecs; ++u) to[base + (int64_t)u * kMoveThreads] = buf[u];
    }
    return;
  }
  // ragged last chunk of a slot
  for (int64_t v = first; v < slot_vecs; v += kMoveThreads) to[v] = __builtin_nontemporal_load(from + v);
}

// Moves that only the backup can serve, where it is in host memory: kLinkBlocks workgroups take 4 KiB of them in turn.  Bound by
// the host link, which wants few requests in flight: 28.3 MB in one launch of 64 KiB to a workgroup, all of it asked for
// at once, take 558 us (50.7 GB/s); a vector per thread of 32 / 64 / 128 / 256 / 512 / 1024 workgroups 502 / 500 / 504 / 503 / 509 / 544,
// four of 64 / 256 503 / 542, eight of 16 / 64 / 256 504 / 510 / 549; the copy engine 508.  Whole calls, a full grid / these: 8 experts
// of 1 MB 50.3 / 55.7 GB/s, 6 and 12 of 4.7 MB 51.5 and 53.6 / 56.9 and 57.2, 7 of 18.9 MB 55.0 / 57.5, 7 and 14 of 44 MB 55.6 and
// 55.8 / 57.5 and 57.6.  (A move whose peer has dropped out meanwhile is seen on the GPU only, and takes the backup's copy at the full
// grid's rate.)
constexpr int kLinkBlocks = 64;
__device__ __forceinline__ void copy_over_link(u32x4* weights, const u32x4* backup, int64_t slot_vecs, int block,
                                               const int32_t* mv_dst, const int32_t* mv_expert, int n) {
  const int64_t tiles = (slot_vecs + kMoveThreads - 1) / kMoveThreads;  // of a move
  int m = 0;
  for (int64_t tile = block; m < n; tile += kLinkBlocks) {
    while (tile >= tiles) {
      tile -= tiles;
      if (++m == n) return;
    }
    const int64_t v = tile * kMoveThreads + threadIdx.x;
    if (v < slot_vecs)
      weights[mv_dst[m] * slot_vecs + v] = __builtin_nontemporal_load(backup + mv_expert[m] * slot_vecs + v);
  }
}

// The mask as it stands now, not as it stood when the plan was made; only the
// source is looked up (a destination may belong to a rank that has not joined yet).
__device__ __forceinline__ bool is_from_peer(int src, const int32_t* active, int S) {
  return src >= 0 && active[src / S] != 0;
}
__device__ __forceinline__ int outcome_of(int src, bool from_peer) {
  return from_peer ? EEP_REPAIR_FROM_PEER : src >= 0 ? EEP_REPAIR_FROM_DRAM_FALLBACK : EEP_REPAIR_FROM_DRAM;
}

// One workgroup's part of the moves.  Of n moves the last n_link go over the host link, by the first kLinkBlocks workgroups (if
// there are any); each of the others copies one chunk, a move's chunks one after the other.  The outcome of a move is
// written by whoever copies its first vectors, from the look at the mask that chose their source: one of its own would be at
// another time, and another context's combine may drop the rank in between.
__device__ __forceinline__ void move_weights(int block, u32x4* weights, const u32x4* backup, int64_t slot_vecs,
                                             int chunks_per_move, const int32_t* mv_dst, const int32_t* mv_src,
                                             const int32_t* mv_expert, int n, int n_link, const int32_t* active, int S,
                                             int32_t* outcome) {
  if (n_link > 0) {
    if (block < kLinkBlocks) {
      const int first = n - n_link;
      if (block == 0)
        for (int m = first + threadIdx.x; m < n; m += kMoveThreads) outcome[mv_dst[m]] = EEP_REPAIR_FROM_DRAM;
      copy_over_link(weights, backup, slot_vecs, block, mv_dst + first, mv_expert + first, n_link);
      return;
    }
    block -= kLinkBlocks;
  }
  const int m = block / chunks_per_move, chunk = block - m * chunks_per_move;
  const int src = mv_src[m], dst = mv_dst[m];
  const bool from_peer = is_from_peer(src, active, S);
  if (chunk == 0 && threadIdx.x == 0) outcome[dst] = outcome_of(src, from_peer);
  copy_chunk(weights, backup, slot_vecs, chunk, dst, src, mv_expert[m], from_peer);
}

__global__ __launch_bounds__(kMoveThreads) void k_relocate(
    u32x4* weights, const u32x4* backup, int64_t slot_vecs, int chunks_per_move, int n, int n_link,
    const int32_t* __restrict__ mv_dst, const int32_t* __restrict__ mv_src,
    const int32_t* __restrict__ mv_expert, const int32_t* __restrict__ active, int S,
    int32_t* __restrict__ outcome) {
  move_weights(blockIdx.x, weights, backup, slot_vecs, chunks_per_move, mv_dst, mv_src, mv_expert, n, n_link, active, S,
               outcome);
}

// The whole repair in one launch, where its move list and the new tables fit the kernel's arguments: workgroup 0 writes the
// tables and the outcomes of slots that nothing moves to (nothing in the launch reads these, and what comes behind it on
// the stream sees both them and the weights), the others move.  Bound by the copies; a launch for the move list and one for the tables cost some 2.2 us each
// (a repair, a return with 28 MB over the host link and the way back to the preferred placement: 593.7 us with
// them, 582.6 without, 530.0 with few workgroups on the link).
constexpr int kRepairInts = 960, kRepairSmallInts = 320;
template <int N>
struct RepairWords {  // of n moves the destinations, the sources, the experts; slot -> expert [P], list starts [E+1], lists [P]
  int32_t v[N];
};

template <int N>
__global__ __launch_bounds__(kMoveThreads) void k_repair(
    u32x4* weights, const u32x4* backup, int64_t slot_vecs, int chunks_per_move, int n, int n_link, int S,
    const int32_t* active, int P, int E, int32_t* outcome, int32_t* p2l, int32_t* l2p_off, int32_t* l2p_list,
    int32_t* version, RepairWords<N> words) {
  const int32_t* mv_dst = words.v;
  const int32_t *mv_src = mv_dst + n, *mv_expert = mv_src + n, *tables = mv_expert + n;
  if (blockIdx.x > 0) {
    move_weights(blockIdx.x - 1, weights, backup, slot_vecs, chunks_per_move, mv_dst, mv_src, mv_expert, n, n_link,
                 active, S, outcome);
    return;
  }
  __shared__ int32_t s_moved[N];
  for (int p = threadIdx.x; p < P; p += kMoveThreads) s_moved[p] = 0;
  __syncthreads();
  for (int m = threadIdx.x; m < n; m += kMoveThreads) s_moved[mv_dst[m]] = 1;
  for (int i = threadIdx.x; i < 2 * P + E + 1; i += kMoveThreads) {
    const int32_t v = tables[i];
    if (i < P) p2l[i] = v;
    else if (i < P + E + 1) l2p_off[i - P] = v;
    else l2p_list[i - P - E - 1] = v;
  }
  __syncthreads();
  for (int p = threadIdx.x; p < P; p += kMoveThreads)
    if (s_moved[p] == 0) outcome[p] = EEP_REPAIR_UNTOUCHED;
  if (threadIdx.x == 0) *version = *version + 1;
}

template <int N>
hipError_t launch_repair(eep_ctx* c, u32x4* weights, const u32x4* backup, int64_t slot_vecs, int chunks, int blocks,
                         const std::vector<int32_t>& words, int n, int n_link, hipStream_t st) {
  RepairWords<N> w;
  memcpy(w.v, words.data(), words.size() * sizeof(int32_t));
  memset(w.v + words.size(), 0, (N - words.size()) * sizeof(int32_t));
  hipLaunchKernelGGL(k_repair<N>, dim3((unsigned)blocks), dim3(kMoveThreads), 0, st, weights, backup, slot_vecs,
                     chunks, n, n_link, c->S, c->active, c->P, c->E, c->mv_outcome, c->p2l, c->l2p_off, c->l2p_list,
                     c->tbl_version, w);
  return hipGetLastError();
}

int fail_hip(eep_ctx* c, hipError_t e) {
  c->last_hip_error = (int)e;
  return EEP_ERR_HIP;
}

// Is [p, p + bytes) GPU-readable memory of the kind the contract names?  On
// success *dev_ptr is the address a kernel uses, and *on_host whether it is host memory.
bool gpu_readable(const void* p, int64_t bytes, bool device_only, int device, const void** dev_ptr,
                  bool* on_host = nullptr) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const bool on_device = at.type == hipMemoryTypeDevice && at.device == device;
  const bool pinned_host = at.type == hipMemoryTypeHost && !device_only && at.devicePointer != nullptr;
  if (!on_device && !pinned_host) return false;
  // the enclosing allocation must contain the whole range
  void* base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange((hipDeviceptr_t*)&base, &size, (hipDeviceptr_t)p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if ((const char*)p + bytes > (const char*)base + size) return false;
  *dev_ptr = p;  // pinned host memory is mapped at its host address
  if (on_host != nullptr) *on_host = pinned_host;
  return true;
}

}  // namespace

extern "C" {

int eep_apply_repair(eep_ctx* c, void* weights, const void* backup, int64_t slot_bytes,
                     const int32_t* new_p2l, const int32_t* kind, const int32_t* src_slot,
                     void* stream) {
  if (!c || !weights || !new_p2l || !kind || !src_slot || slot_bytes <= 0)
    return EEP_ERR_INVALID_ARG;
  if (slot_bytes % 16 != 0 || ((uintptr_t)weights & 15u) || ((uintptr_t)backup & 15u))
    return EEP_ERR_ALIGN;
  c = c->tables;  // a staging context names its owner's tables
  const int P = c->P, S = c->S;
  std::vector<int32_t> dst, src, expert, link_dst, link_expert;  // (those that only the backup serves come last)
  for (int p = 0; p < P; ++p) {
    const int e = new_p2l[p];
    if (e < -1 || e >= c->E) return EEP_ERR_INVALID_ARG;
    switch (kind[p]) {
      case EEP_SRC_NONE:
        break;
      case EEP_SRC_LOCAL:
        if (e < 0 || c->h_p2l[p] != e) return EEP_ERR_INVALID_ARG;
        break;
      case EEP_SRC_PEER: {
        const int q = src_slot[p];
        if (e < 0 || q < 0 || q >= P || q == p || c->h_p2l[q] != e) return EEP_ERR_INVALID_ARG;
        if (kind[q] == EEP_SRC_PEER || kind[q] == EEP_SRC_DRAM) return EEP_ERR_INVALID_ARG;
        dst.push_back(p); src.push_back(q); expert.push_back(e);
        break;
      }
      case EEP_SRC_DRAM:
        if (e < 0) return EEP_ERR_INVALID_ARG;
        link_dst.push_back(p); link_expert.push_back(e);
        break;
      default:
        return EEP_ERR_INVALID_ARG;
    }
  }
  // Sources are looked up in the device mask per transfer, so an unread detection round
  // does not matter for the movement; the coverage check of a strict context does need a
  // current mask.
  if (c->cfg.strict_coverage) {
    if (c->mem->unread_round) return EEP_ERR_STATE;
    if (host_uncovered_experts(P, c->E, S, new_p2l, c->mem->h_active.data()) > 0)
      return EEP_ERR_COVERAGE;
  }
  dst.insert(dst.end(), link_dst.begin(), link_dst.end());
  src.insert(src.end(), link_dst.size(), -1);
  expert.insert(expert.end(), link_expert.begin(), link_expert.end());
  const int n_moves = (int)dst.size();
  const int64_t slot_vecs = slot_bytes / 16;
  const int64_t chunks = (slot_vecs + kChunkVecs - 1) / kChunkVecs;
  if ((int64_t)n_moves * chunks > 0x7fffffffLL) return EEP_ERR_INVALID_ARG;
  const void* weights_dev = nullptr;
  const void* backup_dev = nullptr;
  bool backup_on_host = false;
  if (!gpu_readable(weights, (int64_t)P * slot_bytes, true, c->device, &weights_dev))
    return EEP_ERR_INVALID_ARG;
  if (n_moves > 0) {
    if (!backup) return EEP_ERR_INVALID_ARG;
    if (!gpu_readable(backup, (int64_t)c->E * slot_bytes, false, c->device, &backup_dev, &backup_on_host))
      return EEP_ERR_INVALID_ARG;
  }

  hipStream_t st = (hipStream_t)stream;
  hipError_t e;
  const int n_link = backup_on_host ? (int)link_dst.size() : 0;
  const int64_t blocks = (n_link > 0 ? kLinkBlocks : 0) + (n_moves - n_link) * chunks;  // that move
  const int64_t n_words = (int64_t)3 * n_moves + 2 * (int64_t)P + c->E + 1;
  if (n_words <= kRepairInts) {
    // (what publish_placement checks has been checked above)
    std::vector<int32_t> words(n_words);
    std::copy(dst.begin(), dst.end(), words.begin());
    std::copy(src.begin(), src.end(), words.begin() + n_moves);
    std::copy(expert.begin(), expert.end(), words.begin() + 2 * n_moves);
    int32_t* const tables = words.data() + 3 * n_moves;
    std::copy(new_p2l, new_p2l + P, tables);
    host_replica_lists(P, c->E, S, c->S_prim, new_p2l, tables + P, tables + P + c->E + 1);
    const auto launch = n_words <= kRepairSmallInts ? launch_repair<kRepairSmallInts> : launch_repair<kRepairInts>;
    e = launch(c, (u32x4*)weights_dev, (const u32x4*)backup_dev, slot_vecs, (int)chunks, (int)blocks + 1, words, n_moves,
               n_link, st);
    if (e != hipSuccess) return fail_hip(c, e);
    c->h_p2l.assign(new_p2l, new_p2l + P);
    return EEP_OK;
  }
  // the move list, with every slot's outcome set to "untouched" in the same launch
  e = launch_patch({{c->mv_dst, dst.data(), n_moves},
                    {c->mv_src, src.data(), n_moves},
                    {c->mv_expert, expert.data(), n_moves}},
                   nullptr, st, c->mv_outcome, P, EEP_REPAIR_UNTOUCHED);
  if (e == hipSuccess && n_moves > 0) {
    k_relocate<<<dim3((unsigned)blocks), dim3(kMoveThreads), 0, st>>>(
        (u32x4*)weights_dev, (const u32x4*)backup_dev, slot_vecs, (int)chunks, n_moves, n_link, c->mv_dst,
        c->mv_src, c->mv_expert, c->active, S, c->mv_outcome);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return fail_hip(c, e);
  return publish_placement(c, new_p2l, true, st);
}

int eep_read_repair_outcome(eep_ctx* c, int32_t* outcome_host) {
  if (!c || !outcome_host) return EEP_ERR_INVALID_ARG;
  c = c->tables;  // the repair ran on the tables' owner, whichever context was named
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess)
    e = hipMemcpy(outcome_host, c->mv_outcome, sizeof(int32_t) * (size_t)c->P, hipMemcpyDeviceToHost);
  return e == hipSuccess ? EEP_OK : fail_hip(c, e);
}

}  // extern "C"
