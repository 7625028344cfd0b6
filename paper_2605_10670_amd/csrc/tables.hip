// In-place table patching (paper Sec. 4.1 "In-place peer-table updates",
// Fig. 4, Fig. 8): the tables live at fixed device addresses; an update is a
// tiny kernel that carries the new contents BY VALUE in its kernel arguments,
// so no host buffer has to outlive the call and nothing is allocated, copied
// through staging memory or synchronised.
#include <string.h>

#include "eep_internal.hpp"

namespace eep {

// One launch carries up to kPatchInts (or, for a short update, kPatchSmallInts) values of up
// to kPatchParts arrays that lie end to end in `chunk`; `first` is how many values of the
// whole update came in earlier launches.  fill_n words at fill_dst get fill_value.
// version_dst (may be null): a word that counts the changes of the table; it is bumped on
// the device, so that changes made by kernels (a rank dropped by the waiting kernel) and
// changes made by the host share one count.
// An update of a placement at 32 x 9 slots (833 words) is one launch this way; with one launch
// per array and 2 KB each it was three of about 2 us on the GPU and 3 us of host time.
constexpr int kPatchThreads = 256;
template <int N>
struct PatchChunk {
  int32_t v[N];
};
struct PatchDst {
  int32_t* dst[kPatchParts];
  int32_t end[kPatchParts];  // of the array's values in the whole update
};

template <int N>
__global__ __launch_bounds__(kPatchThreads) void k_patch(int32_t* dst0, int32_t* dst1, int32_t* dst2, int32_t* version_dst,
                                                         int end0, int end1, int first, int n, int fill_n,
                                                         int32_t fill_value, int32_t* fill_dst, PatchChunk<N> chunk) {
  // Bound by latency: the values, which need none of the arguments before them, and the old version are on their way at
  // once (a placement of 32 x 9 slots 2.2 us on the GPU, 3.9 with a wait in each round of the loop; an empty kernel takes 1.9)
  constexpr int kEach = (N + kPatchThreads - 1) / kPatchThreads;
  const int tid = threadIdx.x;
  int32_t v[kEach];
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    const int i = tid + u * kPatchThreads;
    v[u] = chunk.v[i < N ? i : N - 1];
  }
  const int32_t version = version_dst != nullptr && tid == 0 ? *version_dst : 0;
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    const int i = tid + u * kPatchThreads, at = first + i;
    if (i >= n) break;
    if (at < end0) dst0[at] = v[u];
    else if (at < end1) dst1[at - end0] = v[u];
    else dst2[at - end1] = v[u];
  }
  for (int i = tid; i < fill_n; i += kPatchThreads) fill_dst[i] = fill_value;
  if (version_dst != nullptr && tid == 0) *version_dst = version + 1;
}

__global__ __launch_bounds__(256) void k_fill(int32_t* __restrict__ dst, int32_t value, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) dst[i] = value;
}

template <int N>
static hipError_t launch_patch_chunk(const PatchDst& to, const PatchArray* parts, int first, int n,
                                     int32_t* fill_dst, int fill_n, int32_t fill_value,
                                     int32_t* version_dst, hipStream_t st) {
  PatchChunk<N> chunk;
  int begin = 0, done = 0;  // where array q begins in the update; values copied
  for (int q = 0; q < kPatchParts; ++q) {
    const int lo = first + done - begin;
    int m = to.end[q] - begin - lo;
    if (m > n - done) m = n - done;
    if (m > 0) {
      memcpy(&chunk.v[done], parts[q].src + lo, (size_t)m * sizeof(int32_t));
      done += m;
    }
    begin = to.end[q];
  }
  for (int i = done; i < N; ++i) chunk.v[i] = 0;
  hipLaunchKernelGGL(k_patch<N>, dim3(1), dim3(kPatchThreads), 0, st, to.dst[0], to.dst[1], to.dst[2], version_dst,
                     to.end[0], to.end[1], first, n, fill_n, fill_value, fill_dst, chunk);
  return hipGetLastError();
}

hipError_t launch_patch(const PatchArray (&parts)[kPatchParts], int32_t* version_dst, hipStream_t st,
                        int32_t* fill_dst, int fill_n, int32_t fill_value) {
  PatchDst to;
  int total = 0;
  for (int q = 0; q < kPatchParts; ++q) {
    total += parts[q].n;
    to.dst[q] = parts[q].dst;
    to.end[q] = total;
  }
  int done = 0;
  do {
    const int m = total - done < kPatchInts ? total - done : kPatchInts;
    // The version word is bumped by the last chunk, after the data it describes; the fill
    // goes with the first.
    int32_t* version = done + m == total ? version_dst : nullptr;
    const int fill = done == 0 ? fill_n : 0;
    hipError_t e =
        m <= kPatchSmallInts
            ? launch_patch_chunk<kPatchSmallInts>(to, parts, done, m, fill_dst, fill, fill_value, version, st)
            : launch_patch_chunk<kPatchInts>(to, parts, done, m, fill_dst, fill, fill_value, version, st);
    if (e != hipSuccess) return e;
    done += m;
  } while (done < total);
  return hipSuccess;
}

hipError_t launch_fill(int32_t* dst, int32_t value, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)blocks), dim3(256), 0, st, dst, value, n);
  return hipGetLastError();
}

}  // namespace eep
