// Small host-device transfers in one launch each.
//
// A call on a few small frames moves a dozen arrays of some hundred bytes: poses, tables, results.  As one copy each
// they cost more than the kernels between them (3.5 us per copy to the device, 20 us per copy to pageable memory,
// which also waits).  The values of an upload travel as the argument of a kernel that writes them to their
// destinations (3.2 us for all of them, and the host memory is free again at once); a download is a kernel that
// gathers every piece into pinned host memory, waited for once (11 us).
#include "rkhsba_device.h"

namespace rkhsba {
namespace {

constexpr int kThreads = 256;

template <int WORDS>
struct PutArgs {
  uint32_t* dst[kMaxPieces];
  int32_t end[kMaxPieces];  // first word of the payload behind the piece's
  uint32_t w[WORDS];
};

template <int WORDS>
__global__ __launch_bounds__(kThreads) void k_put(PutArgs<WORDS> a) {
  int begin = 0;
  for (int k = 0; k < kMaxPieces; ++k) {
    for (int i = begin + (int)threadIdx.x; i < a.end[k]; i += kThreads) a.dst[k][i - begin] = a.w[i];
    begin = a.end[k];
  }
}

struct GetArgs {
  const uint32_t* src[kMaxPieces];
  int32_t item[kMaxPieces], count[kMaxPieces];  // words per item, items
  int64_t stride[kMaxPieces];                   // words from one item to the next
};

__global__ __launch_bounds__(kThreads) void k_get(GetArgs a, uint32_t* __restrict__ out) {
  for (int k = 0; k < kMaxPieces; ++k) {
    const int n = a.item[k] * a.count[k];
    for (int i = threadIdx.x; i < n; i += kThreads) {
      const int c = i / a.item[k];
      out[i] = a.src[k][c * a.stride[k] + (i - c * a.item[k])];
    }
    out += n;
  }
}

template <int WORDS>
hipError_t put(const Upload* up, int n, hipStream_t st) {
  PutArgs<WORDS> a;
  int words = 0;
  for (int k = 0; k < kMaxPieces; ++k) {
    a.dst[k] = k < n ? static_cast<uint32_t*>(up[k].dst) : nullptr;
    if (k < n && up[k].bytes) {
      std::memcpy(a.w + words, up[k].src, up[k].bytes);
      words += (int)(up[k].bytes / 4);
    }
    a.end[k] = words;
  }
  k_put<WORDS><<<1, kThreads, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace

bool put_fits(const Upload* up, int n) {
  if (n > kMaxPieces) return false;
  size_t total = 0;
  for (int k = 0; k < n; ++k) {
    if (up[k].bytes % 4) return false;
    total += up[k].bytes;
  }
  return total <= kPutBytes;
}

hipError_t launch_put(const Upload* up, int n, hipStream_t st) {
  if (!put_fits(up, n)) return hipErrorInvalidValue;
  size_t total = 0;
  for (int k = 0; k < n; ++k) total += up[k].bytes;
  if (total == 0) return hipSuccess;
  return total <= 256 ? put<64>(up, n, st) : put<kPutBytes / 4>(up, n, st);
}

hipError_t launch_get(const Download* dn, int n, void* pinned, hipStream_t st) {
  if (n > kMaxPieces) return hipErrorInvalidValue;
  GetArgs a{};
  for (int k = 0; k < n; ++k) {
    if (dn[k].item % 4 || dn[k].stride % 4 || dn[k].item * dn[k].count > kGetBytes) return hipErrorInvalidValue;
    a.src[k] = static_cast<const uint32_t*>(dn[k].src);
    a.item[k] = (int32_t)(dn[k].item / 4);
    a.count[k] = (int32_t)dn[k].count;
    a.stride[k] = (int64_t)(dn[k].stride / 4);
  }
  k_get<<<1, kThreads, 0, st>>>(a, static_cast<uint32_t*>(pinned));
  return hipGetLastError();
}

}  // namespace rkhsba
