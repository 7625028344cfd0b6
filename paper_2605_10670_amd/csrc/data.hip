// The bandwidth-bound half of the step: pack (dispatch), the expert stand-ins,
// and the weighted gather-reduce (combine).
//
// Paper: Fig. 7 (dispatch writes one token row per (token, destination)),
// Sec. 4.1 (combine reduces the expert outputs), Sec. 6.2 (dispatch and
// combine dominate the cost of EP serving).  Nothing here is a contraction:
// every kernel is bound by HBM traffic, so the design rules are 16-byte
// accesses, whole 64-lane wavefronts on contiguous 1 KiB spans, each input byte
// read once, and enough independent loads in flight per lane.
#include <type_traits>

#include "eep_internal.hpp"
#include "rows.hpp"

namespace eep {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// pack: recv[row_of[t, j]] = x[t].  One wavefront per token reads the row once
// into registers (up to kPackVecs 16-byte vectors per lane per pass, every load
// issued before the first store) and stores it to the token's k rows; each
// store instruction covers 1 KiB of contiguous row.  Measured on MI355X at the
// decode shape: fatter workgroups, persistent grids, column-split tokens and
// destination-ordered (gather) forms were all slower; stores marked
// write-through at system scope were ~5 % faster than plain or non-temporal
// stores.
// ---------------------------------------------------------------------------
constexpr int kPackVecs = 14;
constexpr int kRowBatch = 8;  // row indices fetched together
// Batches below this many tokens split a row over wavefronts, and below the second many, and those of few bytes (pack_split),
// in pieces as narrow as combine's.  Counts of tokens, where they were checked (rows of 0.5, 1,
// 2, 4, 5.6, 8, 14 and 16 KiB and fp32 rows of 8 and 32 KiB, T = 32 to 4096, identity and scaling
// experts) no step is more than 1 % slower than with 2 KiB pieces below 1024 tokens and 2 KiB parts
// in combine, and most are faster.
constexpr int kPackSplitBelow = 1024;
constexpr int kPackNarrowBelow = 512;
constexpr int kExpandSplitBelow = 4096;  // the same for rows that are read and written once

// One wavefront per token.  U = 16-byte vectors per lane per pass.  EXACT: the row is a whole number of
// passes (row_vecs % (64 * U) == 0), so no access needs a bounds check;
// otherwise loads past the row's end read its last vector again, so that all U
// loads of a pass are in flight here too (a branch around each would make it
// wait for the ones before), and stores are guarded.
template <int U, bool EXACT>
__global__ __launch_bounds__(64) void k_pack(const u32x4* __restrict__ x,
                                             const int32_t* __restrict__ row_of, int k,
                                             int row_vecs, u32x4* __restrict__ recv) {
  const int t = blockIdx.x;
  const int lane = threadIdx.x;
  const int32_t* rows = row_of + (int64_t)t * k;
  const u32x4* src = x + (int64_t)t * row_vecs;
  for (int v0 = 0; v0 < row_vecs; v0 += 64 * U) {
    u32x4 buf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int v = v0 + u * 64 + lane;
      if (!EXACT && v >= row_vecs) v = row_vecs - 1;
      buf[u] = __builtin_nontemporal_load(&src[v]);
    }
    // Touch every loaded register here, so that the waits for the loads sit in
    // front of the row loop and the stores of consecutive rows stream out
    // without a wait between them.
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" ::"v"(buf[u]));
    for (int j = 0; j < k; ++j) {
      int row = rows[j];
      if (row < 0) continue;
      u32x4* dst = recv + (int64_t)row * row_vecs;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int v = v0 + u * 64 + lane;
        if (EXACT || v < row_vecs) store_row(&dst[v], buf[u]);
      }
    }
  }
}

// Small batches, which would leave most of the chip idle that way: one wavefront per piece of 64 * U
// vectors of a token's row, and for fp8 payloads (SCALES) one more for its scale row.  Bound by
// latency, that is by the instructions of a wavefront, some 5 cycles each, and by the launch: k is a
// compile-time number up to kSplitMaxK, whose row indices are one scalar load, the data load comes
// before them, and a store takes its row from a scalar address.  Measured on whole steps in a graph of 8
// (7168 channels, top-8): T = 32 / 256 in 10.2 / 21.5 us with 5 scalar instructions to an index and 18 to
// a store, 10.05 / 21.35 now; with fp8 payloads, whose scale rows were a launch of their own behind
// (k_scale_rows), T = 32 / 128 / 512 / 1000 in 16.3 / 19.9 / 42.4 / 70.7 us, 13.2 / 17.2 / 38.6 / 67.0 now.
constexpr int kSplitMaxK = 8;

template <int U, bool EXACT, int K, bool SCALES>
__global__ __launch_bounds__(64) void k_pack_split(const u32x4* __restrict__ x,
                                                   const int32_t* __restrict__ row_of, int k_rt,
                                                   uint32_t row_vecs, uint32_t parts, uint32_t magic,
                                                   u32x4* __restrict__ recv,
                                                   const u32x4* __restrict__ x_scale,
                                                   u32x4* __restrict__ recv_scale, uint32_t scale_vecs) {
  const int k = K > 0 ? K : k_rt;
  const uint32_t t = token_of(blockIdx.x, parts, magic);
  const uint32_t part = blockIdx.x - t * parts, lane = threadIdx.x;
  const int32_t* rows = row_of + (int64_t)t * k;
  // f(row) for the token's rows, with the data in `touch` waited for ahead of the first, so that no
  // store waits for the one before
  const auto for_rows = [&](auto touch, auto f) {
    if constexpr (K > 0) {
      int r[K];
#pragma unroll
      for (int j = 0; j < K; ++j) r[j] = rows[j];
      touch();
#pragma unroll
      for (int j = 0; j < K; ++j)
        if (r[j] >= 0) f(r[j]);
    } else {
      for (int j0 = 0; j0 < k; j0 += kRowBatch) {
        int r[kRowBatch];
#pragma unroll
        for (int i = 0; i < kRowBatch; ++i) r[i] = rows[j0 + i < k ? j0 + i : k - 1];
        touch();
#pragma unroll
        for (int i = 0; i < kRowBatch; ++i)
          if (j0 + i < k && r[i] >= 0) f(r[i]);
      }
    }
  };
  if (SCALES && part == parts - 1) {  // the scale row, a vector per lane and pass
    for (uint32_t v0 = 0; v0 < scale_vecs; v0 += 64) {
      const uint32_t v = v0 + lane < scale_vecs ? v0 + lane : scale_vecs - 1;
      const u32x4 d = x_scale[(int64_t)t * scale_vecs + v];
      for_rows([&]() { asm volatile("" ::"v"(d)); }, [&](int row) {
        if (v0 + lane < scale_vecs)
          store_row_at(recv_scale, (int64_t)row * (scale_vecs * 16), v * 16, d);
      });
    }
    return;
  }
  const u32x4* src = x + (int64_t)t * row_vecs;
  const uint32_t v0 = part * (64 * U) + lane;
  u32x4 buf[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    uint32_t v = v0 + u * 64;
    if (!EXACT && v >= row_vecs) v = row_vecs - 1;
    buf[u] = __builtin_nontemporal_load(&src[v]);
  }
  for_rows([&]() {
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" ::"v"(buf[u]));
  }, [&](int row) {
    // (a row of 4 GiB and more, which the general k takes, is 64 bits of bytes)
    const int64_t at = K > 0 ? (int64_t)row * (row_vecs * 16) : ((int64_t)row * row_vecs + (v0 - lane)) * 16;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (EXACT || v0 + u * 64 < row_vecs)
        store_row_at(recv, at, ((K > 0 ? v0 : lane) + u * 64) * 16, buf[u]);
  });
}

// Several tokens per wavefront: all TPW * U loads of the wavefront are issued
// before its first store, then the TPW * k rows stream out.  Measured on MI355X
// (T = 16384, 7 KiB rows): 212 us with one token per wavefront, 201 with four,
// 192 with eight; what counts is that the launch comes down to about 2048
// wavefronts -- two per SIMD, all resident at once, every load of the launch in
// flight before the stores start.  Fewer wavefronts than that, or a loop over
// token groups inside a wavefront, are slower again.  T % TPW == 0, rows exact.
template <int U, int TPW>
__global__ __launch_bounds__(64) void k_pack_multi(const u32x4* __restrict__ x,
                                                   u32x4* __restrict__ recv,
                                                   const int32_t* __restrict__ row_of, int k,
                                                   int row_vecs) {
  const int t0 = blockIdx.x * TPW;
  const int lane = threadIdx.x;
  u32x4 buf[TPW][U];
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const u32x4* src = x + (int64_t)(t0 + q) * row_vecs;
#pragma unroll
    for (int u = 0; u < U; ++u) buf[q][u] = __builtin_nontemporal_load(&src[u * 64 + lane]);
  }
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
#pragma unroll
    for (int u = 0; u < U; ++u) asm volatile("" ::"v"(buf[q][u]));  // waits sit before the stores
  }
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int32_t* rows = row_of + (int64_t)(t0 + q) * k;
    for (int j = 0; j < k; ++j) {
      int row = rows[j];
      if (row < 0) continue;
      u32x4* dst = recv + (int64_t)row * row_vecs;
#pragma unroll
      for (int u = 0; u < U; ++u) store_row(&dst[u * 64 + lane], buf[q][u]);
    }
  }
}

// Scale rows of fp8 payloads (H/group fp32 values per row; 224 bytes at the
// prefill shape), written in DESTINATION order: a thread owns one 16-byte
// vector of the receive scale buffer, finds the token behind its row through
// src_of, and copies the vector from the small [T][H/group] source table (3.6 MB
// at T = 16384, read 8 times, from cache).  All stores are contiguous.
// Measured at T = 16384 inside the step (payload, scales, combine in a loop):
// token-ordered scatter with one token per wavefront +27 us, with four tokens
// per wavefront +20 us, this form +10 us, for 33 MB; 224-byte rows scattered
// among the payload's write stream are what is expensive there, not the launch; in small batches,
// where it is the launch, k_pack_split moves them.
constexpr int kScaleThreads = 256;
constexpr int kScaleVecs = 4;  // vectors per thread, each an independent chain of lookups
                               // (measured at T = 16384: 2 per thread -1.5 us, 4 -3 us, 8 +5 us
                               // against one vector per thread)

// max_vecs = T * k * scale_vecs (every row the buffers hold), first: the launch's first one; the rows of this
// step end at status[0], which is read beside the first lookups rather than ahead of them.  row_magic: for
// the vector's row, as in token_of, 0 where there are too many vectors for it.
template <int K>
__global__ __launch_bounds__(kScaleThreads) void k_scale_rows(
    const u32x4* __restrict__ x_scale, u32x4* __restrict__ recv_scale,
    const int32_t* __restrict__ src_of, const int32_t* __restrict__ status, int k_rt,
    uint32_t scale_vecs, uint32_t row_magic, int64_t max_vecs) {
  const uint32_t k = K > 0 ? K : k_rt;
  const int64_t v0 = (int64_t)blockIdx.x * (kScaleThreads * kScaleVecs) + threadIdx.x;
  int pair[kScaleVecs];
  uint32_t col[kScaleVecs];
#pragma unroll
  for (int u = 0; u < kScaleVecs; ++u) {
    const int64_t v = v0 + u * kScaleThreads < max_vecs ? v0 + u * kScaleThreads : max_vecs - 1;
    const uint32_t row = row_magic != 0 ? __umulhi((uint32_t)v, row_magic) : (uint32_t)(v / scale_vecs);
    col[u] = (uint32_t)v - row * scale_vecs;
    pair[u] = src_of[row];
  }
  const int64_t n_vecs = (int64_t)status[0] * scale_vecs;  // rows >= N are left untouched
  u32x4 val[kScaleVecs];
#pragma unroll
  for (int u = 0; u < kScaleVecs; ++u) {
    if (v0 + u * kScaleThreads >= n_vecs) pair[u] = -1;
    if (pair[u] >= 0) val[u] = x_scale[(int64_t)((uint32_t)pair[u] / k) * scale_vecs + col[u]];
  }
#pragma unroll
  for (int u = 0; u < kScaleVecs; ++u)
    if (pair[u] >= 0) store_row(&recv_scale[v0 + u * kScaleThreads], val[u]);
}

// How a row of row_vecs 16-byte vectors is cut into passes of 64 * u vectors, and over how many
// wavefronts.  Large batches: one wavefront per token with the largest pass <= max_vecs that
// divides the row (a whole 14 KiB row per wavefront at the decode shape); a row with no such
// pass of at least half that width takes the fewest even passes and checks its end.  `split` > 0 (small
// batches, which would leave most of the chip idle that way): a row is spread over wavefronts,
// each taking one pass of `split` vectors per lane.  Pack below 512 tokens takes 1, the pieces
// that combine reads: workgroups go to the XCDs in turn, so the piece that combine's wavefront
// (token, part) reads is one that the same XCD's pack wrote, where combine reads the receive
// buffer itself.  Measured (7168 channels, identity experts, one set of buffers, a graph of 8
// steps; T = 128 / 256 / 512): 12.4 / 18.9 / 29.2 us with 1, 16.5 / 24.3 / 31.7 with 2; with a set of
// buffers per step 8 steps of 32 / 256 tokens 77.8 / 159.4 against 79.2 / 159.5.  From 512 tokens on
// it is 2, and combine takes its pieces in pairs so that they meet in an XCD again (k_combine):
// with 1 and a scaling stage between (512 tokens, 2048 fp32 channels, top-2) a step takes 22.4 us
// against 19.2.
// Measured on whole steps with rows that are no whole number of passes (bf16, 2880 channels,
// 360 vectors; T = 32 / 256 / 2048): 26 / 30 / 52 us with a bounds check around each of 14
// accesses and one wavefront per token at every T, 9.3 / 15.7 / 42.7 us in this form.
//
// Larger batches of few bytes keep the pieces that combine reads too: the receive rows are then still in the L2s when it
// does.  Measured as whole steps in graphs of 4, the time without over that with narrow pieces: combine reads the receive rows,
// by their MiB, top-4 to 8 of 512 to 3072 tokens 8 1.04-1.08, 12 1.06-1.13, top-2 and 3 of up to 6 MiB of tokens 1.02-1.16, of
// more 0.95-1.04, top-1 0.97-1.04, top-10 (run-time top-k) 0.94; with a kernel between that writes other rows for combine to read
// 0.99-1.03, but 0.95-0.99 from 16 MiB on for top-4 to 8 (where the other gives 1.03-1.17).
static int pack_split_of_tokens(int T) { return T < kPackNarrowBelow ? 1 : T < kPackSplitBelow ? 2 : 0; }
static int pack_split(const eep_ctx* c, int T) {
  const int64_t x_bytes = T * c->x_row_bytes;
  const bool narrow = c->cfg.x_dtype != EEP_FP8_E4M3 && c->k >= 2 && c->k <= kSplitMaxK && x_bytes <= 6 << 20 &&
                      (c->k < 4 || x_bytes * c->k <= 14 << 20);
  return narrow ? 1 : pack_split_of_tokens(T);
}
struct PassShape {
  int u, parts;
  bool exact;
};
static PassShape pass_shape(int row_vecs, int split, int64_t rows, int max_vecs) {
  const int per_lane = (row_vecs + 63) / 64;
  PassShape s = {1, 1, row_vecs % 64 == 0};
  if (split > 0 && per_lane > 1) {
    s.u = split;
    s.exact = row_vecs % (64 * split) == 0;
    s.parts = (per_lane + split - 1) / split;
    if (rows * s.parts <= max_blocks(64)) return s;  // (else the grid would not fit: do not split)
    s = {1, 1, row_vecs % 64 == 0};
  }
  const int passes = (per_lane + max_vecs - 1) / max_vecs;
  const int even = (per_lane + passes - 1) / passes;
  if (s.exact) {
    s.u = max_vecs;
    while (per_lane % s.u != 0) --s.u;
    if (s.u * 2 > even) return s;
  }
  s.u = even;
  s.exact = false;
  return s;
}

template <int U, bool EXACT>
static hipError_t launch_pack_t(eep_ctx* c, const int32_t* rows, const void* x, void* recv_x,
                                int T, hipStream_t st) {
  hipLaunchKernelGGL((k_pack<U, EXACT>), dim3(T), dim3(64), 0, st, (const u32x4*)x, rows, c->k,
                     (int)(c->x_row_bytes / 16), (u32x4*)recv_x);
  return hipGetLastError();
}

template <int U, bool EXACT, bool SCALES>
static hipError_t launch_pack_split_t(eep_ctx* c, const int32_t* rows, const void* x,
                                      const float* x_scale, void* recv_x, float* recv_scale, int T,
                                      int parts, hipStream_t st) {
  static const decltype(&k_pack_split<U, EXACT, 0, SCALES>) of[kSplitMaxK + 1] = {
      k_pack_split<U, EXACT, 0, SCALES>, k_pack_split<U, EXACT, 1, SCALES>,
      k_pack_split<U, EXACT, 2, SCALES>, k_pack_split<U, EXACT, 3, SCALES>,
      k_pack_split<U, EXACT, 4, SCALES>, k_pack_split<U, EXACT, 5, SCALES>,
      k_pack_split<U, EXACT, 6, SCALES>, k_pack_split<U, EXACT, 7, SCALES>,
      k_pack_split<U, EXACT, 8, SCALES>};
  const int64_t grid = (int64_t)T * parts;
  const bool compiled = c->k <= kSplitMaxK && c->x_row_bytes < (int64_t)1 << 32;  // (32-bit offsets there)
  hipLaunchKernelGGL(of[compiled ? c->k : 0], dim3((unsigned)grid), dim3(64), 0, st,
                     (const u32x4*)x, rows, c->k, (uint32_t)(c->x_row_bytes / 16), (uint32_t)parts,
                     part_magic(parts, grid), (u32x4*)recv_x, (const u32x4*)x_scale,
                     (u32x4*)recv_scale, (uint32_t)(c->scale_row_bytes / 16));
  return hipGetLastError();
}

template <int U, int TPW>
static hipError_t launch_pack_multi_t(eep_ctx* c, const int32_t* rows, const void* x, void* recv_x,
                                      int T, hipStream_t st) {
  hipLaunchKernelGGL((k_pack_multi<U, TPW>), dim3(T / TPW), dim3(64), 0, st, (const u32x4*)x,
                     (u32x4*)recv_x, rows, c->k, (int)(c->x_row_bytes / 16));
  return hipGetLastError();
}

// Below 8192 tokens one wavefront per token already fits the chip in one round (8192
// resident wavefronts), and at the decode shape (T = 4096, 14 KiB rows) two tokens per
// wavefront made the step 3 us slower: pack itself no faster, the combine after it slower.
constexpr int kPackMultiMinTokens = 8192;
constexpr int kPackMultiMinWaves = 2048;  // two wavefronts per SIMD of the 256 CUs
constexpr int kPackMultiMaxVecs = 56;     // 16-byte vectors a lane holds at once

// Tokens per wavefront: several in very large batches (>= kPackMultiMinTokens) of whole-row
// passes, as many as keep >= kPackMultiMinWaves wavefronts and <= kPackMultiMaxVecs vectors per lane.
static int pack_tokens_per_wave(const PassShape& ps, int row_vecs, int T) {
  int tpw = 1;
  if (ps.exact && ps.u * 64 == row_vecs)
    while (T >= kPackMultiMinTokens && tpw < 8 && T % (tpw * 2) == 0 &&
           T / (tpw * 2) >= kPackMultiMinWaves && ps.u * tpw * 2 <= kPackMultiMaxVecs)
      tpw *= 2;
  return tpw;
}

// (x_scale null: no scale rows, or not here)
static hipError_t launch_pack_payload(eep_ctx* c, const int32_t* rows, const void* x,
                                      const float* x_scale, void* recv_x, float* recv_scale, int T,
                                      int split, hipStream_t st) {
  const int row_vecs = (int)(c->x_row_bytes / 16);
  const PassShape ps = pass_shape(row_vecs, split, T, kPackVecs);
  if (x_scale != nullptr || ps.parts > 1) {
#define EEP_PACK_SPLIT(U, SCALES)                                                                 \
  return ps.exact ? launch_pack_split_t<U, true, SCALES>(c, rows, x, x_scale, recv_x, recv_scale, \
                                                         T, ps.parts + SCALES, st)                \
                  : launch_pack_split_t<U, false, SCALES>(c, rows, x, x_scale, recv_x, recv_scale, \
                                                          T, ps.parts + SCALES, st)
    if (x_scale != nullptr) {
      if (ps.u == 1) EEP_PACK_SPLIT(1, true);
      EEP_PACK_SPLIT(2, true);
    }
    if (ps.u == 1) EEP_PACK_SPLIT(1, false);
    EEP_PACK_SPLIT(2, false);
#undef EEP_PACK_SPLIT
  }
  const int tpw = pack_tokens_per_wave(ps, row_vecs, T);
  if (tpw > 1) {
    switch (tpw * 16 + ps.u) {
#define EEP_PACK_MULTI(TPW, U) \
  case TPW * 16 + U: return launch_pack_multi_t<U, TPW>(c, rows, x, recv_x, T, st);
      EEP_PACK_MULTI(2, 1) EEP_PACK_MULTI(2, 2) EEP_PACK_MULTI(2, 3) EEP_PACK_MULTI(2, 4)
      EEP_PACK_MULTI(2, 5) EEP_PACK_MULTI(2, 6) EEP_PACK_MULTI(2, 7) EEP_PACK_MULTI(2, 8)
      EEP_PACK_MULTI(2, 9) EEP_PACK_MULTI(2, 10) EEP_PACK_MULTI(2, 11) EEP_PACK_MULTI(2, 12)
      EEP_PACK_MULTI(2, 13) EEP_PACK_MULTI(2, 14)
      EEP_PACK_MULTI(4, 1) EEP_PACK_MULTI(4, 2) EEP_PACK_MULTI(4, 3) EEP_PACK_MULTI(4, 4)
      EEP_PACK_MULTI(4, 5) EEP_PACK_MULTI(4, 6) EEP_PACK_MULTI(4, 7) EEP_PACK_MULTI(4, 8)
      EEP_PACK_MULTI(4, 9) EEP_PACK_MULTI(4, 10) EEP_PACK_MULTI(4, 11) EEP_PACK_MULTI(4, 12)
      EEP_PACK_MULTI(4, 13) EEP_PACK_MULTI(4, 14)
      EEP_PACK_MULTI(8, 1) EEP_PACK_MULTI(8, 2) EEP_PACK_MULTI(8, 3) EEP_PACK_MULTI(8, 4)
      EEP_PACK_MULTI(8, 5) EEP_PACK_MULTI(8, 6) EEP_PACK_MULTI(8, 7)
#undef EEP_PACK_MULTI
    }
  }
  switch (ps.u) {
#define EEP_PACK_CASE(U)                                                                \
  case U:                                                                               \
    return ps.exact ? launch_pack_t<U, true>(c, rows, x, recv_x, T, st)                 \
                    : launch_pack_t<U, false>(c, rows, x, recv_x, T, st);
    EEP_PACK_CASE(14) EEP_PACK_CASE(13) EEP_PACK_CASE(12) EEP_PACK_CASE(11) EEP_PACK_CASE(10)
    EEP_PACK_CASE(9) EEP_PACK_CASE(8) EEP_PACK_CASE(7) EEP_PACK_CASE(6) EEP_PACK_CASE(5)
    EEP_PACK_CASE(4) EEP_PACK_CASE(3) EEP_PACK_CASE(2) EEP_PACK_CASE(1)
#undef EEP_PACK_CASE
  }
  return hipErrorInvalidValue;
}

static hipError_t launch_pack_any(eep_ctx* c, const int32_t* rows, const void* x,
                                  const float* x_scale, void* recv_x, float* recv_scale, int T,
                                  int split, hipStream_t st) {
  if (T == 0) return hipSuccess;
  // Small batches: the scale rows go with the payload, in wavefronts of their own.
  const bool together = x_scale != nullptr && T < kPackSplitBelow &&
                        pass_shape((int)(c->x_row_bytes / 16), split, T, kPackVecs).u <= 2;
  hipError_t e = in_launches(T, max_blocks(64), [&](int64_t t0, int64_t n) {
    return launch_pack_payload(c, rows + t0 * c->k, (const char*)x + t0 * c->x_row_bytes,
                               together ? x_scale : nullptr, recv_x, recv_scale, (int)n, split, st);
  });
  if (e != hipSuccess || x_scale == nullptr || together) return e;
  const int scale_vecs = (int)(c->scale_row_bytes / 16);
  const int64_t vecs = (int64_t)T * c->k * scale_vecs;
  const int64_t per_block = (int64_t)kScaleThreads * kScaleVecs;
  const int64_t blocks = (vecs + per_block - 1) / per_block;
  if (blocks > max_blocks(kScaleThreads)) return hipErrorInvalidValue;
  // (row = v * magic >> 32 is exact while vecs * scale_vecs < 2^32)
  const uint32_t magic = scale_vecs > 1 ? part_magic(scale_vecs, vecs) : 0;
  hipLaunchKernelGGL((c->k == 8 ? k_scale_rows<8> : k_scale_rows<0>), dim3((unsigned)blocks),
                     dim3(kScaleThreads), 0, st, (const u32x4*)x_scale, (u32x4*)recv_scale, c->src_of,
                     c->status, c->k, (uint32_t)scale_vecs, magic, vecs);
  return hipGetLastError();
}

// With the layout in one launch the narrow pieces are the better ones up to larger sizes, also where another kernel writes what
// combine reads (top-8, T = 1024 to 1536 of 1024 channels, 16 to 24 MiB of receive rows: 1.17-1.20 times as fast as two launches,
// 1.09-1.12 with wider pieces; with a scaling stage 1.03-1.10 and 1.02-1.10).  Whether stores are held is for the call that
// reads the rows to say (hold_rows in api.hip).
bool pack_pieces(const eep_ctx* c, const void* x, const float* x_scale, void* recv_x, float* recv_scale, int T,
                 PackPieces* out) {
  const int row_vecs = (int)(c->x_row_bytes / 16), scale_vecs = x_scale != nullptr ? (int)(c->scale_row_bytes / 16) : 0;
  // (scale rows of larger batches are a launch of their own; a piece holds 64 vectors of one)
  if (scale_vecs > 64 || (scale_vecs > 0 && T >= kPackSplitBelow) || c->x_row_bytes >= (int64_t)1 << 32) return false;
  const int chunks = (row_vecs + 63) / 64;
  const int64_t x_bytes = T * c->x_row_bytes;
  int vecs = pack_split(c, T);
  if (scale_vecs == 0 && c->k >= 2 && x_bytes <= 6 << 20 && x_bytes * c->k <= 36 << 20) vecs = 1;
  if (vecs == 0) {  // (whole rows): as few parts as 7 vectors per lane allow
    const int parts = (chunks + 6) / 7, even = (chunks + parts - 1) / parts;
    vecs = even <= 2 ? even : even <= 4 ? 4 : 7;
  }
  *out = {x, x_scale, recv_x, recv_scale, (uint32_t)row_vecs, (uint32_t)scale_vecs,
          (uint32_t)((chunks + vecs - 1) / vecs + (scale_vecs > 0)), vecs, false};
  return true;
}

hipError_t launch_pack(eep_ctx* c, const void* x, const float* x_scale, void* recv_x,
                       float* recv_scale, int T, hipStream_t st) {
  return launch_pack_any(c, c->row_of, x, x_scale, recv_x, recv_scale, T, pack_split(c, T), st);
}

hipError_t launch_pack_rows(eep_ctx* c, const int32_t* rows, const void* x, void* recv, int T,
                            hipStream_t st) {
  return launch_pack_any(c, rows, x, nullptr, recv, nullptr, T, pack_split_of_tokens(T), st);
}

// ---------------------------------------------------------------------------
// Expansion on the destination of a de-duplicated dispatch:
// recv[row] = recv_d[expand_of[row]] for the N routed rows (expand_of is -1 from N
// on).  Bound by HBM like pack, with one store per load.  Below 8192 rows, which
// is what the chip holds in wavefronts, a wavefront has up to 7 vectors per lane in
// flight (T = 512, 5760-byte rows, whole step: 38.8 us, with 2 40.1); from there on
// 2, which keeps the running copies closer to address order (T = 2048, 14 KiB rows:
// 158.5 us, with 4 160, 7 166.7, 14 168.8, and with each pass in a wavefront of its
// own 172).  Rows beyond 16 KiB are many such passes one after the other, and there 8
// are better (32 KiB rows, T = 1024 / 2048 / 4096: 208 / 398 / 810 us, with 2 222 / 403 /
// 820, 4 211 / 401 / 815, 7 with a bounds check 216 / 401 / 813).  Few rows are split like a
// small batch in pack.
// ---------------------------------------------------------------------------
constexpr int kExpandVecs = 7, kExpandManyVecs = 2, kExpandWideVecs = 8;
constexpr int kExpandManyRows = 8192, kExpandWideRow = 16384 / 16;

template <int U, bool EXACT, bool HELD>
__global__ __launch_bounds__(64) void k_expand(const int32_t* __restrict__ expand_of,
                                               const u32x4* __restrict__ recv_d, int row_vecs,
                                               uint32_t parts, uint32_t magic,
                                               u32x4* __restrict__ recv) {
  const int row = token_of(blockIdx.x, parts, magic);
  const int from = expand_of[row];
  if (from < 0) return;  // rows past the last routed pair
  const u32x4* src = recv_d + (int64_t)from * row_vecs;
  u32x4* dst = recv + (int64_t)row * row_vecs;
  for (int v0 = (blockIdx.x - row * parts) * 64 * U + threadIdx.x; v0 < row_vecs;
       v0 += parts * 64 * U) {
    u32x4 buf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int v = v0 + u * 64;
      if (!EXACT && v >= row_vecs) v = row_vecs - 1;
      buf[u] = __builtin_nontemporal_load(&src[v]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (EXACT || v0 + u * 64 < row_vecs) store_row<HELD>(&dst[v0 + u * 64], buf[u]);
  }
}

hipError_t launch_expand(eep_ctx* c, const void* recv_dedup, void* recv_x, int T, hipStream_t st, hipGraphNode_t held) {
  const int64_t rows = (int64_t)T * c->k;
  if (rows == 0) return hipSuccess;
  const int row_vecs = (int)(c->x_row_bytes / 16);
  const PassShape ps = pass_shape(row_vecs, rows < kExpandSplitBelow ? 2 : 0, rows,
                                  rows < kExpandManyRows       ? kExpandVecs
                                  : row_vecs <= kExpandWideRow ? kExpandManyVecs
                                                               : kExpandWideVecs);
  return in_launches(rows, max_blocks(64) / ps.parts, [&](int64_t r0, int64_t n) {
    const int32_t* expand_of = c->dd_expand + r0;
    const u32x4* from = (const u32x4*)recv_dedup;
    int vecs = row_vecs;
    uint32_t parts = (uint32_t)ps.parts, magic = part_magic(ps.parts, n * ps.parts);
    u32x4* to = (u32x4*)recv_x + r0 * row_vecs;
    const unsigned grid = (unsigned)(n * ps.parts);
    void* args[] = {&expand_of, &from, &vecs, &parts, &magic, &to};
    switch (ps.u) {
#define EEP_EXPAND_CASE(U)                                                                                      \
  case U:                                                                                                       \
    if (held != nullptr) {                                                                                      \
      const auto kern = ps.exact ? k_expand<U, true, true> : k_expand<U, false, true>;                          \
      return set_node(held, (const void*)kern, grid, 64, 0, args) ? hipSuccess : hipErrorInvalidValue;          \
    }                                                                                                           \
    hipLaunchKernelGGL((ps.exact ? k_expand<U, true, false> : k_expand<U, false, false>), dim3(grid), dim3(64), \
                       0, st, expand_of, from, vecs, parts, magic, to);                                         \
    return hipGetLastError();
      EEP_EXPAND_CASE(8) EEP_EXPAND_CASE(7) EEP_EXPAND_CASE(6) EEP_EXPAND_CASE(5) EEP_EXPAND_CASE(4)
      EEP_EXPAND_CASE(3) EEP_EXPAND_CASE(2) EEP_EXPAND_CASE(1)
#undef EEP_EXPAND_CASE
    }
    return hipErrorInvalidValue;
  });
}

// ---------------------------------------------------------------------------
// number formats
// ---------------------------------------------------------------------------
__device__ inline float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// Two binary32 -> two bfloat16 in one dword, round to nearest even, NaN stays (quiet) NaN: one
// v_cvt_pk_bf16_f32.  Compared with the integer form of the rule (add 0x7fff and the kept
// bit, shift) over all 2^32 inputs, NaNs and subnormals included: no difference.
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// binary32 -> OCP e4m3fn byte, round to nearest even, saturating at +-448
// (NaN -> 0x7f).  Normal results round the 23-bit significand to 3 bits with an
// integer add so that a carry moves into the exponent; results below 2^-6 are
// multiples of 2^-9.
__device__ inline uint32_t f32_to_e4m3(float f) {
  uint32_t u = __float_as_uint(f);
  uint32_t sign = (u >> 24) & 0x80u;
  uint32_t a = u & 0x7fffffffu;
  if (a > 0x7f800000u) return sign | 0x7fu;      // NaN
  if (a >= 0x43e00000u) return sign | 0x7eu;     // |f| >= 448: saturate
  uint32_t code;
  if (a < 0x3c800000u) {                         // |f| < 2^-6: subnormal range
    float scaled = __uint_as_float(a) * 512.0f;  // exact; in [0, 8)
    code = (uint32_t)__float2int_rn(scaled);     // ties to even; 8 is the smallest normal
  } else {
    uint32_t r = a + 0x7ffffu + ((a >> 20) & 1u);
    code = (r >> 20) - ((127u - 7u) << 3);
    if (code > 0x7eu) code = 0x7eu;              // 448 < |f| rounded past the top
  }
  return sign | code;
}

// ---------------------------------------------------------------------------
// pack with quantisation fused in (a data-path variant the paper's Sec. 4.1
// leaves to prior work): x is bf16, the receive rows are e4m3 codes plus one
// fp32 scale per `group` channels.  Per token and group: scale = max|x| / 448
// (1 if the group is all zero), code = e4m3(x / scale).  A lane owns 16
// consecutive channels (32 bytes in, 16 bytes out), so the lanes of a group are
// neighbours and the group maximum is a few lane exchanges.  The token is
// quantised once and stored to its k rows.  Large batches: one wavefront per
// token, 7 vectors per lane; below kQuantSplitBelow tokens a wavefront per 64
// vectors, for latency.
//
// The store stream is the bound, and the arithmetic stands in front of it: all
// wavefronts of a launch load, then compute, then store, so vector instructions
// are not hidden.  Hence, per channel, four of them instead of a division and an
// integer conversion (some 25): with y = 1 / scale correctly rounded and
// q = x * y, the residual r = x - q * scale is exact in one fused multiply-add
// and q + r * y is the correctly rounded quotient (P. W. Markstein, "Computation
// of elementary functions on the IBM RISC System/6000 processor", IBM J. Res.
// Dev. 34, 1990) while nothing under- or overflows; v_cvt_pk_fp8_f32 rounds it.
// Compared with the division and f32_to_e4m3 for EVERY pair of a finite bf16
// maximum with its scale in [2^-100, 2^100] and a bf16 x up to it, both signs: no
// code differs.  (Of the 444,868,577 pairs of one sign 1,023,886 have another quotient, all with
// |x| < 2^-43, from residuals or quotients that underflow; it rounds to the same code.)  Groups
// outside (infinities and NaN among them) take the division.
// Measured, whole step with the dequantising stand-in (7168 channels, T = 32 / 256 / 4096):
// 28.1 / 40.5 / 248 us before, 15.7 / 29.8 / 254 split by size but with divisions and with the scale
// stores among the rows, 14.4 / 28.1 / 242.5 now.
// ---------------------------------------------------------------------------
constexpr int kQuantVecs = 7;           // 16-channel vectors per lane per pass (7 * 64 * 16 = 7168)
constexpr int kQuantSplitBelow = 1024;  // batches below this many tokens split a row over wavefronts

// Maximum over aligned groups of n lanes (n a power of two <= 64), in every lane of the group.
__device__ __forceinline__ uint32_t group_max(uint32_t v, int n) {
  auto larger = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  if (n > 1) v = larger(v, __builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xf, 0xf, false));   // lane ^ 1
  if (n > 2) v = larger(v, __builtin_amdgcn_update_dpp(0u, v, 0x4E, 0xf, 0xf, false));   // lane ^ 2
  if (n > 4) v = larger(v, __builtin_amdgcn_update_dpp(0u, v, 0x141, 0xf, 0xf, false));  // half row mirrored
  if (n > 8) v = larger(v, __builtin_amdgcn_update_dpp(0u, v, 0x140, 0xf, 0xf, false));  // row mirrored
  for (int m = 16; m < n; m <<= 1) v = larger(v, __shfl_xor(v, m, 64));
  return v;
}

__device__ __forceinline__ uint32_t quant4(const uint32_t (&d)[2], float scale, float y) {
  float q[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float x = i & 1 ? bf16_hi(d[i >> 1]) : bf16_lo(d[i >> 1]);
    const float q0 = x * y;
    const float r = fmaf(-q0, scale, x);
    q[i] = copysignf(fmaf(r, y, q0), x);  // (a zero keeps its sign)
  }
  int o = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], o, true);
}

template <int U>
__global__ __launch_bounds__(64) void k_pack_quant(const u32x4* __restrict__ x,
                                                   const int32_t* __restrict__ row_of, int k,
                                                   int out_vecs, uint32_t parts, uint32_t magic,
                                                   int lanes_per_group, int groups,
                                                   u32x4* __restrict__ recv_q,
                                                   float* __restrict__ recv_scale) {
  __shared__ float s_scale[U * 64];  // scales of this pass
  const int t = token_of(blockIdx.x, parts, magic);
  const int lane = threadIdx.x;
  const bool leader = (lane & (lanes_per_group - 1)) == 0;
  const int log_lanes = __builtin_ctz(lanes_per_group);
  const int32_t* rows = row_of + (int64_t)t * k;
  const u32x4* src = x + (int64_t)t * out_vecs * 2;
  for (int w0 = (blockIdx.x - t * parts) * 64 * U; w0 < out_vecs; w0 += parts * 64 * U) {
    u32x4 in[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // past the row's end: its last vector again; groups are whole, so no group with a lane
      // before the end has one behind it
      int w = w0 + u * 64 + lane;
      if (w >= out_vecs) w = out_vecs - 1;
      in[u][0] = __builtin_nontemporal_load(&src[2 * w]);
      in[u][1] = __builtin_nontemporal_load(&src[2 * w + 1]);
    }
    u32x4 q[U];
    uint32_t odd = 0;  // bit u: this lane's group of vector u needs the division
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // magnitudes of bf16 compare as integers, two at a time; NaN above everything
      u16x2 m2 = {0, 0};
#pragma unroll
      for (int i = 0; i < 8; ++i)
        m2 = __builtin_elementwise_max(
            m2, __builtin_bit_cast(u16x2, in[u][i >> 2][i & 3] & 0x7fff7fffu));
      const uint32_t top = group_max(m2[0] > m2[1] ? m2[0] : m2[1], lanes_per_group);
      float scale = __uint_as_float(top << 16) / 448.0f;
      if (scale == 0.0f) scale = 1.0f;
      if (top >= 0x7f80u || scale < 0x1p-100f || scale > 0x1p100f) odd |= 1u << u;
      if (leader) s_scale[(u * 64 + lane) >> log_lanes] = scale;
      const float y = 1.0f / scale;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t d[2] = {in[u][i >> 1][2 * (i & 1)], in[u][i >> 1][2 * (i & 1) + 1]};
        q[u][i] = quant4(d, scale, y);
      }
    }
    for (int j = 0; j < k; ++j) {
      int row = rows[j];
      if (row < 0) continue;
      u32x4* dst = recv_q + (int64_t)row * out_vecs;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int w = w0 + u * 64 + lane;
        if (w < out_vecs) store_row(&dst[w], q[u]);
      }
    }
    if (__any(odd != 0)) {
      // rare: the groups in question once more, from memory, one vector at a time; what was
      // stored for them above is complete before it is overwritten
      __threadfence();
      for (int u = 0; u < U; ++u) {
        const int w = w0 + u * 64 + lane;
        if (((odd >> u) & 1u) == 0 || w >= out_vecs) continue;
        float v[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t d = src[2 * w + (i >> 2)][i & 3];
          v[2 * i] = bf16_lo(d);
          v[2 * i + 1] = bf16_hi(d);
        }
        float amax = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(v[i]));
        for (int m = 1; m < lanes_per_group; m <<= 1) amax = fmaxf(amax, __shfl_xor(amax, m, 64));
        float scale = amax / 448.0f;
        if (scale == 0.0f) scale = 1.0f;
        if (leader) s_scale[(u * 64 + lane) >> log_lanes] = scale;
        u32x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          o[i] = f32_to_e4m3(v[4 * i] / scale) | (f32_to_e4m3(v[4 * i + 1] / scale) << 8) |
                 (f32_to_e4m3(v[4 * i + 2] / scale) << 16) |
                 (f32_to_e4m3(v[4 * i + 3] / scale) << 24);
        for (int j = 0; j < k; ++j)
          if (rows[j] >= 0) store_row(&recv_q[(int64_t)rows[j] * out_vecs + w], o);
      }
    }
    __syncthreads();
    const int g0 = w0 >> log_lanes;
    for (int g = lane; g < (U * 64) >> log_lanes && g0 + g < groups; g += 64) {
      const float sc = s_scale[g];
      for (int j = 0; j < k; ++j) {
        int row = rows[j];
        if (row >= 0) recv_scale[(int64_t)row * groups + g0 + g] = sc;
      }
    }
    __syncthreads();
  }
}

hipError_t launch_pack_quant(eep_ctx* c, const void* x_bf16, void* recv_q, float* recv_scale, int T,
                             hipStream_t st) {
  if (T == 0) return hipSuccess;
  const int out_vecs = c->H / 16;
  const int groups = c->H / c->cfg.scale_group;
  const int passes = (out_vecs + 63) / 64;
  const bool split = T < kQuantSplitBelow && (int64_t)T * passes <= max_blocks(64);
  const int parts = split ? passes : 1;
  return in_launches(T, max_blocks(64) / parts, [&](int64_t t0, int64_t n) {
    hipLaunchKernelGGL((split ? k_pack_quant<1> : k_pack_quant<kQuantVecs>),
                       dim3((unsigned)(n * parts)), dim3(64), 0, st,
                       (const u32x4*)x_bf16 + t0 * out_vecs * 2, c->row_of + t0 * c->k, c->k,
                       out_vecs, (uint32_t)parts, part_magic(parts, n * parts),
                       c->cfg.scale_group / 16, groups, (u32x4*)recv_q, recv_scale);
    return hipGetLastError();
  });
}

// ---------------------------------------------------------------------------
// combine: out[t] = sum_j w[t,j] * y[row_of[t,j]], fp32 fused multiply-add chain
// in ascending j.  A lane owns 16-byte columns of the row and issues the k row
// loads of its columns back to back.
// ---------------------------------------------------------------------------
template <bool Y_BF16>
struct YVec {
  static constexpr int kElems = Y_BF16 ? 8 : 4;
};

template <bool Y_BF16>
__device__ inline void accumulate(float (&acc)[YVec<Y_BF16>::kElems], u32x4 v, float w) {
  if constexpr (Y_BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[2 * i] = fmaf(w, bf16_lo(v[i]), acc[2 * i]);
      acc[2 * i + 1] = fmaf(w, bf16_hi(v[i]), acc[2 * i + 1]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = fmaf(w, __uint_as_float(v[i]), acc[i]);
  }
}

template <bool Y_BF16, bool OUT_BF16>
__device__ inline void store_out(void* out_row, int v, const float (&acc)[YVec<Y_BF16>::kElems]) {
  if constexpr (Y_BF16 && OUT_BF16) {
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(acc[2 * i], acc[2 * i + 1]);
    __builtin_nontemporal_store(o, (u32x4*)out_row + v);
  } else if constexpr (Y_BF16 && !OUT_BF16) {
    f32x4 a = {acc[0], acc[1], acc[2], acc[3]}, b = {acc[4], acc[5], acc[6], acc[7]};
    __builtin_nontemporal_store(a, (f32x4*)out_row + 2 * v);
    __builtin_nontemporal_store(b, (f32x4*)out_row + 2 * v + 1);
  } else if constexpr (!Y_BF16 && OUT_BF16) {
    u32x2 o = {pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3])};
    __builtin_nontemporal_store(o, (u32x2*)out_row + v);
  } else {
    f32x4 a = {acc[0], acc[1], acc[2], acc[3]};
    __builtin_nontemporal_store(a, (f32x4*)out_row + v);
  }
}

// ---------------------------------------------------------------------------
// GPU-side failure detection inside combine (paper Sec. 3.4; Sec. 4.1, the
// paragraph on failure detection from the GPU side): before a wavefront reduces
// a token's rows it looks at the signal word of every rank those rows come
// from.  The expert stage stores the step's epoch there once the rank's outputs
// are in place.  A word that does not show the epoch sends the wavefront into
// the wait below; a rank that stays silent past the time-out is dropped by the
// kernel: its `active` entry is cleared, it is put on the report that the host
// reads after the kernel, the membership version is bumped, and the pairs
// routed to it contribute nothing (their row_of entry becomes -1).
// In a healthy step the first wavefront of the launch finds every expected
// signal in place and publishes that in one word (round_ok = epoch); the others
// read that word (one agent-scope load, issued beside the row indices) and go
// straight on.  Wavefronts that run before the word is published, and all
// wavefronts of a step in which a signal is missing, look at the signals of
// their own rows' ranks, a pair per lane.  No row is loaded before one or the other has
// said that it is there: a signal may come from another stream while the kernel
// runs.  Those first looks use plain loads: they either see the epoch or lead to the wait.
// The wait itself uses agent-scope loads,
// so that a rank dropped by a wavefront on another XCD is seen at once and all
// waiting wavefronts together spend about one time-out, not one each.  Every
// wait is bounded by the wall clock and by a poll count.
// ---------------------------------------------------------------------------
struct DetectArgs {
  const int32_t* slot_of;     // [T, k]
  int32_t* row_of;            // [T, k], entries of dropped pairs are set to -1
  const int32_t* signal;      // [R] epoch of the last step whose outputs arrived
  const int32_t* step_epoch;  // current step
  int32_t* active;            // [R]
  int32_t* report;            // [R]
  int32_t* mem_version;
  const int32_t* rank_count;  // [R] rows each rank holds in this step
  int32_t* round_ok;          // epoch of the last step in which every expected signal was there
  int R, S;
  long long timeout_ticks, max_polls;
};

// pending: bit j set = pair j's rank has not signalled.  Returns the bits of the pairs whose
// rank was dropped (by this wavefront or by another).  Uniform across the wavefront.
__device__ __forceinline__ uint32_t await_late_ranks(const DetectArgs& d, int64_t pair0, uint32_t pending,
                                                  int epoch) {
  uint32_t failed = 0;
  const long long t0 = wall_clock64();
  long long polls = 0;
  while (pending != 0) {
    for (uint32_t m = pending; m != 0; m &= m - 1) {
      const int j = __ffs(m) - 1;
      const int rank = d.slot_of[pair0 + j] / d.S;
      if (__hip_atomic_load(&d.signal[rank], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == epoch) {
        pending &= ~(1u << j);  // arrived late
      } else if (__hip_atomic_load(&d.active[rank], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
        pending &= ~(1u << j);  // dropped meanwhile
        failed |= 1u << j;
      }
    }
    if (pending == 0) break;
    if (++polls > d.max_polls || wall_clock64() - t0 > d.timeout_ticks) {
      // time-out: drop every rank still awaited; the first wavefront to clear the entry
      // also reports it
      for (uint32_t m = pending; m != 0; m &= m - 1) {
        const int j = __ffs(m) - 1;
        const int rank = d.slot_of[pair0 + j] / d.S;
        if (threadIdx.x == 0 &&
            __hip_atomic_exchange(&d.active[rank], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
          __hip_atomic_store(&d.report[rank], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_fetch_add(d.mem_version, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        failed |= 1u << j;
      }
      break;
    }
    __builtin_amdgcn_s_sleep(8);
  }
  if (threadIdx.x == 0)
    for (uint32_t m = failed; m != 0; m &= m - 1) d.row_of[pair0 + __ffs(m) - 1] = -1;
  return failed;
}

// First look (plain loads) at the signals of the ranks a token's rows come from; the wait only
// if one is missing.  Lane j brings the row and slot of pair j (-1: none); returns the row, or
// -1 if its rank was dropped.  The rows are not read again here: another wavefront of the token
// may have struck one meanwhile, and a struck row must be reported, not passed over.
__device__ __forceinline__ int row_if_arrived(const DetectArgs& d, int64_t pair0, int row, int slot,
                                              int epoch) {
  const bool missing = row >= 0 && d.signal[slot / d.S] != epoch;
  const uint32_t pending = (uint32_t)__ballot(missing);  // (k <= 32)
  if (pending == 0) return row;
  const uint32_t dropped = await_late_ranks(d, pair0, pending, epoch);
  return threadIdx.x < 32 && ((dropped >> threadIdx.x) & 1u) ? -1 : row;
}

// One wavefront per (token, part): a part is 64 16-byte columns of the row, 1 KiB of each source
// row, and a lane has the k loads of its column in flight.  Bound by HBM; what the kernel
// itself decides is how soon a wavefront's loads are out, hence the order below: row indices,
// row loads, weights.  Measured on whole steps (8 steps of 32 / 256 tokens, 4 of 4096, one of
// 1024 with 1/32 of the pairs dropped; 7168 channels, top-8): 80.4 / 164.7 / 750 / 51.7 us; with
// two columns per lane 82.6 / 166.4 / 756 / 52.5, four 86.9 / 169 / 763 / 56.7; two columns with a
// bounds check around each column's loads (the second column's then waited for the first's)
// 83.2 / 168 / 755 / 57.  Single-wavefront workgroups measured ~10 % faster than one workgroup
// per token.
//
// `paired` > 0 (the number of tokens): the batch was packed in pieces of two parts (batches of 512
// to 1023 tokens; whole rows of 1 to 2 KiB in larger ones), `parts` counts such pieces, and the
// two wavefronts of piece m run on the XCD that wrote it (workgroups go to the 8 XCDs in turn,
// pack's m-th to m mod 8): 16 workgroups take pieces 8g .. 8g + 7, first their first parts and
// then their second.  Measured (identity experts, one set of buffers, whole steps of T = 512 / 768 /
// 992 tokens): 2048 channels 20.6 / 26.6 / 29.1 us without, 15.4 / 19.0 / 22.1 with; 4096 channels
// 28.0 / 32.1 / 35.7 and 20.5 / 28.5 / 33.5; 7168 channels 32.6 / 42.4 / 51.0 and 29.6 / 40.9 / 49.7;
// 1024 channels, T = 1024 / 2048: 22.0 / 29.2 and 17.0 / 22.9; with a scaling stage between, where
// nothing can meet, within 1 % either way.
//
// k is a compile-time number up to 10; a larger one goes in batches of 8 and 4 rows.  One row at a
// time, each behind its index, top-10 took (whole steps, 4096 channels, T = 32 / 256) 12.5 / 16.9 us instead
// of 9.7 / 15.5, top-3 9.2 / 10.4 instead of 8.7 / 9.9, top-5 of 512 tokens 21.9 instead of 21.1; at 4096
// tokens, where other wavefronts fill the time, 124.8 instead of 123.0 and the same; top-32 of 1024 tokens 43.2 instead
// of 44.7.  With one pair in seven dropped (combine alone, 4096 channels, T = 256 / 1024, top-12 / 24 / 32) one row at a time
// 10.3 / 17.4, 17.3 / 30.6, 21.7 / 39.1 us, a batch with such a pair one row at a time 9.1 / 17.9, 15.7 / 33.0, 19.6 / 42.1,
// a branch around each load 8.2 / 17.8, 15.5 / 33.1, 19.4 / 42.0, and in this form 6.2 / 16.6, 9.0 / 30.3, 11.0 / 39.2.
//
// DETECT: the wait for the ranks' signals is part of the kernel (DetectArgs above); row_of
// is then not read-only, because dropped pairs are struck from it, and lane j keeps the row of
// pair j from the one time it was read.
template <bool Y_BF16, bool OUT_BF16, int K, bool DETECT>
__global__ __launch_bounds__(64) void k_combine(const int32_t* row_of,
                                                const u32x4* __restrict__ y, int k, int row_vecs,
                                                uint32_t parts, uint32_t magic, int paired,
                                                const float* __restrict__ topk_w,
                                                void* __restrict__ out, DetectArgs det) {
  constexpr int NE = YVec<Y_BF16>::kElems;
  int t, v;
  if (paired > 0) {
    const uint32_t piece = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7);
    t = token_of(piece, parts, magic);
    if (t >= paired) return;
    v = ((piece - t * parts) * 2 + ((blockIdx.x >> 3) & 1)) * 64 + threadIdx.x;
  } else {
    t = token_of(blockIdx.x, parts, magic);
    v = (blockIdx.x - t * parts) * 64 + threadIdx.x;
  }
  const int32_t* rows = row_of + (int64_t)t * k;
  const float* ws = topk_w + (int64_t)t * k;
  void* out_row = (char*)out + (int64_t)t * row_vecs * (NE * (OUT_BF16 ? 2 : 4));

  int my_row = -1;  // of pair threadIdx.x, with DETECT
  if constexpr (DETECT) {
    const int64_t pair0 = (int64_t)t * k;
    int my_slot = -1;
    if ((int)threadIdx.x < k) {
      my_row = rows[threadIdx.x];
      my_slot = det.slot_of[pair0 + threadIdx.x];
    }
    const int epoch = *det.step_epoch;
    if (blockIdx.x == 0) {
      // the first wavefront looks at every rank that holds rows of this step
      bool ok = true;
      for (int r = threadIdx.x; r < det.R; r += 64)
        ok &= det.active[r] == 0 || det.rank_count[r] == 0 || det.signal[r] == epoch;
      if (__all(ok) && threadIdx.x == 0)
        __hip_atomic_store(det.round_ok, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__hip_atomic_load(det.round_ok, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch)
      my_row = row_if_arrived(det, pair0, my_row, my_slot, epoch);
  }
  const auto row_at = [&](int j) { return DETECT ? __builtin_amdgcn_readlane(my_row, j) : rows[j]; };
  const bool past_end = v >= row_vecs;
  if constexpr (DETECT) {
    if (past_end) v = row_vecs - 1;  // a lane with a pair's row stays, whatever its column
  } else if (past_end) {
    return;
  }

  float acc[NE];
#pragma unroll
  for (int i = 0; i < NE; ++i) acc[i] = 0.0f;
  if constexpr (K > 0) {
    // compile-time k: all loads are issued before the first is used
    int r[K];
    bool all = true;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      r[j] = row_at(j);
      all &= (r[j] >= 0);
    }
    u32x4 d[K];
    if (__builtin_expect(all, 1)) {  // every pair routed: no branch between loads
#pragma unroll
      for (int j = 0; j < K; ++j)
        d[j] = __builtin_nontemporal_load(&y[(int64_t)r[j] * row_vecs + v]);
      // (the weights are read here: scalar loads return in any order, so a wait for the row
      // indices would also be one for the weights, which come from HBM)
#pragma unroll
      for (int j = 0; j < K; ++j) accumulate<Y_BF16>(acc, d[j], ws[j]);
    } else {
      // Some pairs have no row (a dead rank's experts before the repair, masked indices): the
      // same, with a branch around each load and each term; r[] is uniform, so no lane
      // diverges.  One load at a time here cost 4 us of 57 at T = 1024 with 22 % such tokens.
#pragma unroll
      for (int j = 0; j < K; ++j)
        if (r[j] >= 0) d[j] = __builtin_nontemporal_load(&y[(int64_t)r[j] * row_vecs + v]);
#pragma unroll
      for (int j = 0; j < K; ++j)
        if (r[j] >= 0) accumulate<Y_BF16>(acc, d[j], ws[j]);
    }
  } else {
    const auto batch = [&](auto size, int j0) {
      constexpr int B = decltype(size)::value;
      int r[B];
      bool all = true;
#pragma unroll
      for (int i = 0; i < B; ++i) {
        r[i] = row_at(j0 + i);
        all &= r[i] >= 0;
      }
      u32x4 d[B];
      if (__builtin_expect(all, 1)) {
#pragma unroll
        for (int i = 0; i < B; ++i) d[i] = __builtin_nontemporal_load(&y[(int64_t)r[i] * row_vecs + v]);
#pragma unroll
        for (int i = 0; i < B; ++i) accumulate<Y_BF16>(acc, d[i], ws[j0 + i]);
      } else {
        // Some pairs have no row: they load another one, row 0, or with DETECT one of the token's, which
        // is known to be there, and only the terms are left out.
        int other = 0;
        if constexpr (DETECT) {
          other = -1;
#pragma unroll
          for (int i = 0; i < B; ++i) other = r[i] >= 0 ? r[i] : other;
          if (other < 0) return;
        }
#pragma unroll
        for (int i = 0; i < B; ++i)
          d[i] = __builtin_nontemporal_load(&y[(int64_t)(r[i] >= 0 ? r[i] : other) * row_vecs + v]);
#pragma unroll
        for (int i = 0; i < B; ++i)
          if (r[i] >= 0) accumulate<Y_BF16>(acc, d[i], ws[j0 + i]);
      }
    };
    int j = 0;
    for (; j + 8 <= k; j += 8) batch(std::integral_constant<int, 8>(), j);
    if (j + 4 <= k) {
      batch(std::integral_constant<int, 4>(), j);
      j += 4;
    }
    for (; j < k; ++j) batch(std::integral_constant<int, 1>(), j);
  }
  if (!DETECT || !past_end) store_out<Y_BF16, OUT_BF16>(out_row, v, acc);
}

template <bool Y_BF16, bool OUT_BF16>
static hipError_t launch_combine_t(eep_ctx* c, const void* y, const float* w, void* out, int T,
                                   hipStream_t st) {
  int row_vecs = (int)(c->y_row_bytes / 16);
  int parts = (row_vecs + 63) / 64;
  // (y can be the receive buffer only if its rows are of the same size)
  const int split = c->dispatched_split >= 0 ? c->dispatched_split : pack_split(c, T);
  const PassShape packed = pass_shape(row_vecs, split, T, kPackVecs);
  const bool paired = c->x_row_bytes == c->y_row_bytes && parts > 1 &&
                      (parts + 1) / 2 == packed.parts && pack_tokens_per_wave(packed, row_vecs, T) == 1;
  if (paired) parts = packed.parts;
  DetectArgs det = {};
  const bool detect = c->detect_timeout_ticks > 0;
  if (detect) {
    // the wait for the ranks' signals runs inside the kernel
    det.slot_of = c->slot_of; det.row_of = c->row_of; det.signal = c->signal;
    det.step_epoch = c->step_epoch; det.active = c->active; det.report = c->report;
    det.mem_version = c->mem->mem_version; det.S = c->S; det.R = c->R;
    det.rank_count = c->rank_count; det.round_ok = c->round_ok;
    det.timeout_ticks = c->detect_timeout_ticks;
    det.max_polls = c->detect_timeout_ticks * 8 + 1024;
  }
  // (pairs are rounded up to 8 pieces of two wavefronts)
  const int64_t most = paired ? (max_blocks(64) - 16) / (2 * parts) : max_blocks(64) / parts;
  return in_launches(T, most, [&](int64_t t0, int64_t n) {
    const int64_t pieces = paired ? (n * parts + 7) / 8 * 8 : n * parts;
    const dim3 grid((unsigned)(paired ? 2 * pieces : pieces)), block(64);
    const uint32_t magic = part_magic(parts, pieces);
    const int64_t p0 = t0 * c->k;
    void* to = (char*)out + t0 * c->out_row_bytes;
    DetectArgs d = det;
    if (detect) {
      d.slot_of += p0;
      d.row_of += p0;
    }
    switch (c->k) {
#define EEP_COMBINE_K(CASE, K)                                                              \
  CASE:                                                                                     \
  hipLaunchKernelGGL((detect ? k_combine<Y_BF16, OUT_BF16, K, true>                         \
                             : k_combine<Y_BF16, OUT_BF16, K, false>),                      \
                     grid, block, 0, st, c->row_of + p0, (const u32x4*)y, c->k, row_vecs,   \
                     (uint32_t)parts, magic, paired ? (int)n : 0, w + p0, to, d);           \
  break;
      EEP_COMBINE_K(case 1, 1) EEP_COMBINE_K(case 2, 2) EEP_COMBINE_K(case 3, 3)
      EEP_COMBINE_K(case 4, 4) EEP_COMBINE_K(case 5, 5) EEP_COMBINE_K(case 6, 6)
      EEP_COMBINE_K(case 7, 7) EEP_COMBINE_K(case 8, 8) EEP_COMBINE_K(case 9, 9)
      EEP_COMBINE_K(case 10, 10)
      EEP_COMBINE_K(default, 0)
#undef EEP_COMBINE_K
    }
    return hipGetLastError();
  });
}

hipError_t launch_combine(eep_ctx* c, const void* y, const float* w, void* out, int T,
                          hipStream_t st) {
  if (T == 0) return hipSuccess;
  bool yb = c->cfg.y_dtype == EEP_BF16, ob = c->cfg.out_dtype == EEP_BF16;
  if (yb && ob) return launch_combine_t<true, true>(c, y, w, out, T, st);
  if (yb && !ob) return launch_combine_t<true, false>(c, y, w, out, T, st);
  if (!yb && ob) return launch_combine_t<false, true>(c, y, w, out, T, st);
  return launch_combine_t<false, false>(c, y, w, out, T, st);
}

// ---------------------------------------------------------------------------
// expert stand-ins: what a caller's expert kernels do between dispatch and combine, no
// part of either.  Copy and scale take a workgroup per receive row, with the loads and
// stores of pack (non-temporal, write-through); rows >= N are skipped.  The
// dequantising one is a flat stream of its own, see there.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_stub_copy(const u32x4* __restrict__ recv,
                                                   u32x4* __restrict__ y,
                                                   const int32_t* __restrict__ status,
                                                   int row_vecs, int row0) {
  const int row = row0 + blockIdx.x;
  if (row >= status[0]) return;
  for (int v = threadIdx.x; v < row_vecs; v += blockDim.x)
    store_row(&y[(int64_t)row * row_vecs + v],
              __builtin_nontemporal_load(&recv[(int64_t)row * row_vecs + v]));
}

// y[row] = round(s[expert of row] * recv[row]).  The way to the row's scale is four dependent
// lookups (pair, slot, expert, scale), so the thread's first vector, which needs none of them,
// is on its way meanwhile; a row past N has no pair.  Bound by HBM for large batches; measured, whole
// steps: 764 us against 771 with the row's loads after the lookups (8 steps of 2048 tokens,
// 4096 channels), 11.05 against 11.55 (64 tokens, 2048 channels, top-4).  One wavefront per row or per
// 64 to 512 vectors of one, with non-temporal stores: 787 to 793 (write-through 776), 11.2 to 11.9.
template <bool BF16, bool HELD>
__global__ __launch_bounds__(256) void k_stub_scale(
    const int32_t* __restrict__ src_of, const u32x4* __restrict__ recv, int row_vecs,
    const int32_t* __restrict__ slot_of, const int32_t* __restrict__ p2l,
    const float* __restrict__ expert_scale, u32x4* __restrict__ y) {
  const int row = blockIdx.x;
  const int pair = src_of[row];
  const int64_t base = (int64_t)row * row_vecs;
  int v = threadIdx.x;
  u32x4 d = __builtin_nontemporal_load(&recv[base + (v < row_vecs ? v : row_vecs - 1)]);
  if (pair < 0) return;  // rows >= N are left untouched
  const int e = p2l[slot_of[pair]];
  const float s = e >= 0 ? expert_scale[e] : 0.0f;
  while (v < row_vecs) {
    u32x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (BF16) o[i] = pack_bf16x2(s * bf16_lo(d[i]), s * bf16_hi(d[i]));
      else o[i] = __float_as_uint(s * __uint_as_float(d[i]));
    }
    store_row<HELD>(&y[base + v], o);
    v += 256;
    if (v < row_vecs) d = __builtin_nontemporal_load(&recv[base + v]);
  }
}

// Dequantising stand-in: y = bf16(code * scale).  Receive rows, scale rows and output rows
// are all dense and a scale group never crosses a row (H % group == 0), so the rows [0, N)
// are one flat stream: vector i of 8 codes uses scale i / (group / 8).  Bound by HBM (8 bytes
// in, 16 out per vector): a wavefront reads 512 and writes 1024 contiguous bytes per
// instruction, and the conversions stay out of the way with v_cvt_pk_f32_fp8 (exact), one
// multiply and v_cvt_pk_bf16_f32 (integer conversions of 16 codes per thread, one workgroup
// per row, were bound by the vector ALU: 1228 us for 131072 rows of 7168, now about 450 us = 6.3 TB/s).
// Measured on whole steps (T = 16384 / 4096, H = 7168): 2 vectors per thread 1015 / 252 us, 4
// 1037 / 255, 8 1049 / 255, 16 1110 / 279, 1 1054 / 279; the fewer a block holds, the closer
// to address order the stream runs.  Blocks of 64 threads 1001 / 259, of 512 1026 / 252.
// Non-temporal stores, because nothing is scattered here: write-through stores 1092 / 279,
// plain ones 1085 / 278; plain loads 1086 / 259.
constexpr int kDequantThreads = 256;
constexpr int kDequantVecs = 2;

// Eight codes times one scale.  Code 0x7f is +NaN and 0xff -NaN; the hardware's conversion gives
// both a set sign, which dwords that hold a NaN code (rare) put right.
__device__ __forceinline__ u32x4 dequant8(u32x2 d, float sc) {
  const float nan = __uint_as_float(0x7fc00000u);
  u32x4 o;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)d[i], false);
    f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)d[i], true);
    if ((((d[i] & 0x7f7f7f7fu) + 0x01010101u) & 0x80808080u) != 0) {
      if ((d[i] & 0xffu) == 0x7fu) lo[0] = nan;
      if (((d[i] >> 8) & 0xffu) == 0x7fu) lo[1] = nan;
      if (((d[i] >> 16) & 0xffu) == 0x7fu) hi[0] = nan;
      if ((d[i] >> 24) == 0x7fu) hi[1] = nan;
    }
    o[2 * i] = pack_bf16x2(sc * lo[0], sc * lo[1]);
    o[2 * i + 1] = pack_bf16x2(sc * hi[0], sc * hi[1]);
  }
  return o;
}

// One block's share: kDequantVecs vectors per thread from `q` on, `left` of them exist.  WHOLE:
// all of them, so nothing is guarded and every load is in flight before the first wait.
// `in0`: how far the first vector lies inside the group of the first scale, s0[0].
template <bool POW2, bool WHOLE>
__device__ __forceinline__ void dequant_block(const u32x2* q, const float* s0, u32x4* y,
                                              int64_t left, uint32_t in0, int group_vecs,
                                              int group_shift) {
  const uint32_t tid = threadIdx.x;
  u32x2 d[kDequantVecs];
  float sc[kDequantVecs];
#pragma unroll
  for (int u = 0; u < kDequantVecs; ++u) {
    const uint32_t i = u * kDequantThreads + tid;
    if (WHOLE || i < left) {
      d[u] = __builtin_nontemporal_load(&q[i]);
      sc[u] = s0[POW2 ? (in0 + i) >> group_shift : (in0 + i) / (uint32_t)group_vecs];
    }
  }
#pragma unroll
  for (int u = 0; u < kDequantVecs; ++u) {
    const uint32_t i = u * kDequantThreads + tid;
    if (WHOLE || i < left) __builtin_nontemporal_store(dequant8(d[u], sc[u]), &y[i]);
  }
}

// group_vecs = group / 8; POW2: a power of two, group_shift its logarithm.
template <bool POW2>
__global__ __launch_bounds__(kDequantThreads) void k_stub_dequant(
    const u32x2* __restrict__ q, const float* __restrict__ scale, u32x4* __restrict__ y,
    const int32_t* __restrict__ status, int row_vecs, int group_vecs, int group_shift,
    int64_t block0) {
  const int64_t n = (int64_t)status[0] * row_vecs;  // rows >= N are left untouched
  const int64_t base = (block0 + blockIdx.x) * (kDequantThreads * kDequantVecs);
  if (base >= n) return;
  const int64_t g0 = POW2 ? base >> group_shift
                          : (int64_t)((uint64_t)base / (uint32_t)group_vecs);
  const uint32_t in0 = (uint32_t)(base - g0 * group_vecs);
  if (base + kDequantThreads * kDequantVecs <= n)
    dequant_block<POW2, true>(q + base, scale + g0, y + base, 0, in0, group_vecs, group_shift);
  else
    dequant_block<POW2, false>(q + base, scale + g0, y + base, n - base, in0, group_vecs,
                               group_shift);
}

hipError_t launch_stub(eep_ctx* c, int kind, const void* recv_x, const float* recv_scale,
                       const float* expert_scale, void* y, int T, hipStream_t st) {
  int64_t rows = (int64_t)T * c->k;
  if (rows == 0) return hipSuccess;
  int row_vecs = (int)(c->x_row_bytes / 16);
  const dim3 block(256);
  if (kind != EEP_STUB_DEQUANT)
    return in_launches(rows, max_blocks(256), [&](int64_t r0, int64_t n) {
      const dim3 grid((unsigned)n);
      const int64_t v0 = r0 * row_vecs;
      if (kind == EEP_STUB_IDENTITY) {
        hipLaunchKernelGGL(k_stub_copy, grid, block, 0, st, (const u32x4*)recv_x, (u32x4*)y,
                           c->status, row_vecs, (int)r0);
      } else {
        // Held stores (rows.hpp), in a captured step only: write-through's time over theirs, whole steps, 10-16 / 18 / 24 / 30 MiB:
        // in graphs 1.11-1.18 / 1.08-1.15 / 1.04-1.10 / 1.02-1.04, three sets of buffers in turn 0.99-1.03 / 0.99-1.04 / 1.00-1.03 /
        // 0.98.  Call by call a program may have other buffers each time, and then held stores lose (8 shapes, rows of 2 to 16 KiB,
        // top-2 to 8): one set of buffers, 10-11 / 12 / 14 / 16 MiB 1.02-1.09 / 1.01-1.09 / 1.03-1.13 / 1.06-1.17, two in turn
        // 0.95-1.06 / 0.96-1.05 / 0.97-1.04 / 0.97-1.02, three 0.97-1.01 / 0.97-1.01 / 0.96-1.00 / 0.95-1.00.
        const bool held = mib_between(rows * c->x_row_bytes, 10, 26) && is_captured(st);
        const bool bf16 = c->cfg.x_dtype == EEP_BF16;
        auto kern = held ? (bf16 ? k_stub_scale<true, true> : k_stub_scale<false, true>)
                         : (bf16 ? k_stub_scale<true, false> : k_stub_scale<false, false>);
        hipLaunchKernelGGL(kern, grid, block, 0, st, c->src_of + r0, (const u32x4*)recv_x + v0,
                           row_vecs, c->slot_of, c->p2l, expert_scale, (u32x4*)y + v0);
      }
      return hipGetLastError();
    });
  const int vecs8 = c->H / 8, group_vecs = c->cfg.scale_group / 8;
  const int64_t per_block = kDequantThreads * kDequantVecs;
  const bool pow2 = (group_vecs & (group_vecs - 1)) == 0;
  return in_launches((rows * vecs8 + per_block - 1) / per_block, max_blocks(kDequantThreads),
                     [&](int64_t b0, int64_t n) {
    hipLaunchKernelGGL((pow2 ? k_stub_dequant<true> : k_stub_dequant<false>), dim3((unsigned)n),
                       dim3(kDequantThreads), 0, st, (const u32x2*)recv_x, recv_scale, (u32x4*)y,
                       c->status, vecs8, group_vecs, pow2 ? __builtin_ctz(group_vecs) : 0, b0);
    return hipGetLastError();
  });
}

}  // namespace eep
