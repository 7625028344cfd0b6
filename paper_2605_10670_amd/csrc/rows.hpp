// Device code that every kernel which moves rows shares: pieces of rows, stores.
#pragma once

#include "eep_internal.hpp"

namespace eep {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Workgroup index -> (token, part) without a division in front of the first load: n / d is the
// high word of n * magic, magic = 2^32 / d rounded up, exact while n * d < 2^32 (the rounding
// is at most d too much).  Magic 0: one part, or a grid so large that it divides.
inline uint32_t part_magic(int parts, int64_t grid) {
  if (parts <= 1 || grid * parts >= ((int64_t)1 << 32)) return 0;
  return (uint32_t)((((uint64_t)1 << 32) + parts - 1) / parts);
}
__device__ __forceinline__ uint32_t token_of(uint32_t n, uint32_t parts, uint32_t magic) {
  return magic != 0 ? __umulhi(n, magic) : parts == 1 ? n : n / parts;
}

// Stores of receive rows and of what else one kernel writes and the next one reads, in one of two ways.  Write-through
// (sc0 sc1): a line goes on to memory at once, and stays in the XCD's L2.  HELD (nt): it stays in the L2 until it is
// evicted or the kernel ends, which writes it back.  With the eight L2s of 4 MiB in mind: what fits them is best held, since
// the stores then end in the L2 and the write-back runs at its own pace; larger ones are evicted in the middle of the
// kernel, line by line, and write-through is better; and of a few MB there is nothing to gain, but the write-back at
// the end takes longer than stores that have long arrived.  A buffer whose lines the L2s still hold from the step before gains
// most, one that was not touched lately least: stores that are held then take the place of other lines, and write-through
// ones have no line in another L2 to end.  A captured step is replayed on its own buffers, so stores are held only
// there; calls one by one may have other buffers each time.  The limits at the launches are measured with both.
//
// The data registers of a store of more than 8 bytes may not be rewritten by the next two
// wait states' vector instructions.  The compiler keeps that distance for its own stores but
// does not look into the asm, so the distance is part of it.
template <bool HELD = false>
__device__ __forceinline__ void store_row(u32x4* p, u32x4 v) {
  if constexpr (HELD)
    asm volatile("global_store_dwordx4 %0, %1, off nt\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
  else
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
}

// The same to `offset` bytes behind base + row, both scalar.  A vector memory instruction may not read
// a scalar register within five wait states of a vector instruction that wrote it (v_readfirstlane, or
// a spilled register's v_readlane); the compiler does not keep that distance for asm either, so
// the address is added up by scalar instructions that are part of it.
template <bool HELD = false>
__device__ __forceinline__ void store_row_at(void* base, int64_t row, uint32_t offset, u32x4 v) {
#define EEP_STORE_AT(HOW)                                                                                  \
  asm volatile("s_add_u32 s98, %2, %4\n\ts_addc_u32 s99, %3, %5\n\t"                                       \
               "global_store_dwordx4 %0, %1, s[98:99] " HOW "\n\ts_nop 1" ::"v"(offset), "v"(v),            \
               "s"((uint32_t)(uintptr_t)base), "s"((uint32_t)((uintptr_t)base >> 32)), "s"((uint32_t)row), \
               "s"((uint32_t)((uint64_t)row >> 32))                                                        \
               : "memory", "scc", "s98", "s99")
  if constexpr (HELD)
    EEP_STORE_AT("nt");
  else
    EEP_STORE_AT("sc0 sc1");
#undef EEP_STORE_AT
}

// Makes the captured kernel node one of another launch.
inline bool set_node(hipGraphNode_t node, const void* kernel, unsigned grid, int threads, size_t lds, void** args) {
  hipKernelNodeParams p = {};
  p.func = const_cast<void*>(kernel);
  p.gridDim = dim3(grid);
  p.blockDim = dim3((unsigned)threads);
  p.sharedMemBytes = (unsigned)lds;
  p.kernelParams = args;
  if (hipGraphKernelNodeSetParams(node, &p) == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

// Is a kernel launched on this stream now part of a capture?
inline bool is_captured(hipStream_t st) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (st == nullptr) return false;  // (cannot be)
  if (hipStreamIsCapturing(st, &status) == hipSuccess) return status == hipStreamCaptureStatusActive;
  (void)hipGetLastError();
  return false;
}

// Are `bytes` within [lo, hi] MiB?
inline bool mib_between(int64_t bytes, int lo, int hi) {
  return bytes >= (int64_t)lo << 20 && bytes <= (int64_t)hi << 20;
}

// Does a captured dispatch in one launch with its layout, or a captured expansion, hold its stores of `bytes` of receive rows?  That
// depends on who reads them, and so the call that does, directly behind it, says so.  Write-through's time over that of held stores, whole
// steps in graphs of 4, one / two / three graphs with buffers of their own in turn, by MiB of receive rows of 2 to 14 KiB:
//   combine reads the rows     12 1.03-1.06 / 1.03-1.10 / 1.03-1.07, 16 1.03-1.10 / 1.04-1.11 / 1.01-1.06, 20 1.01-1.18 / 1.01-1.10 /
//                              1.00-1.06, 24 1.00-1.18 / 0.99-1.08 / 0.99-1.03, 28 0.99-1.20 / 0.98-1.05 / 0.97-1.01, 30 to 32 0.97-1.19 /
//                              0.95-1.04 / 0.95-1.00 (rows of 8 KiB gain least: one part of a row is always an XCD's)
//     of an expansion          12 1.02-1.11 / 1.01-1.03 / 1.01-1.05, 16 1.05-1.12 / 1.02-1.04 / 1.01-1.04, 20 1.06-1.11 / 1.01-1.05 /
//                              1.01-1.06, 24 1.02-1.09 / 1.00-1.04 / 1.00-1.05, 28 1.02-1.05 / 0.99-1.02 / 1.00-1.02, 32 1.00-1.05 /
//                              0.99-1.02 / 0.99-1.02
//   the scaling stand-in,      12 1.13-1.17 / 1.01-1.07 / 0.98-1.01, 14 1.12-1.13 / 1.00-1.02 / 0.97-0.98, 16 1.01-1.11 / 0.97-1.00 /
//   which writes others        0.97-0.98, 20 0.98-1.05 / 0.96-1.00 / 0.95-0.98, 24 0.98-0.99 / 0.96-0.97 / 0.95-0.98, 28 1.01 / 1.00 / 1.00
//     of an expansion          12 1.00-1.08 / 0.99-1.06 / 0.99-1.07, 16 to 20 0.98-1.03 / 0.98-1.02 / 0.98-1.02, 24 to 32 0.97-1.00
//   fp8, the dequantising one  4 0.99-1.00 / 1.00-1.03 / 1.02-1.04, 6 0.99-1.03 / 1.03-1.06 / 1.03-1.04, 8 1.04-1.06 / 1.05-1.06 / 1.00-1.03
//   two matrix products        12 to 32 0.98-1.00, whichever (up to 1.2 us a step); an expansion 0.98-1.00; fp8, 4 to 8 0.97-1.00
// The steps of a captured forward pass write one receive buffer in turn, again and again: where the next call of the library reads it,
// the first of the figures decides.  Experts of a program's own read it later and lose, if anything, and nothing is held for them.
// (Against a layout and a dispatch in two launches one gains either way, held 0.99-1.36, write-through 1.00-1.23.  In a dispatch of its
// own, call by call with three sets in turn, held stores lose at every size: 14 / 20 / 26 MiB 0.96-1.06 / 0.97-1.05 / 0.95-1.03, with a
// stage behind it 0.97-0.99 / 0.94-0.98 / 0.93-1.00; quantised, 7 / 9 / 12 MiB of codes 0.98 / 0.95 / 0.92; an expansion, 14 / 18 / 24 / 30
// MiB 0.98-1.00 / 0.98 / 0.94-0.96 / 0.93-0.95.)
enum class RowWriter { kPack, kPackScales, kExpand };
inline bool holds_for_combine(int64_t bytes, RowWriter by) {
  return by == RowWriter::kPack ? mib_between(bytes, 12, 28) : by == RowWriter::kExpand && mib_between(bytes, 12, 32);
}
inline bool holds_for_stub(int64_t bytes, RowWriter by) {
  return by == RowWriter::kPack ? mib_between(bytes, 12, 16) : by == RowWriter::kPackScales && mib_between(bytes, 4, 8);
}

}  // namespace eep
