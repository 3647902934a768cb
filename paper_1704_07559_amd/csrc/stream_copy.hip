// Device copies. The STREAM-style copy is the achievable HBM bandwidth on this device for a pure
// streaming pattern (one read and one write per byte, 16-byte nontemporal accesses, every
// address touched once); the benchmark reports it next to the step kernel, whose roofline is the
// same two streams per population. The state copy moves a context's state (populations and
// rate field) with the same accesses in one launch.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "launch.h"

namespace lbm {

typedef float v4f __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void stream_copy_kernel(const v4f* __restrict__ src, v4f* __restrict__ dst,
                                                          size_t n4) {
  const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n4) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

hipError_t launch_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t st) {
  const size_t n4 = bytes / 16;
  if (n4 == 0) return hipSuccess;
  if (!copy_fits_launch(bytes, 0)) return hipErrorInvalidValue;
  // 5 blocks per CU instead of 8: the copy's own best (6.73 against 6.63 TB/s for 1 GiB; 6 blocks
  // 6.69, 4 blocks 6.38), so that it stays the ceiling the step is compared with
  hipLaunchKernelGGL(stream_copy_kernel, dim3(static_cast<unsigned>(copy_blocks(bytes))), dim3(256),
                     lds_cap_bytes(5, 0), st, static_cast<const v4f*>(src), static_cast<v4f*>(dst), n4);
  return hipGetLastError();
}

// Two ranges, the second one's blocks after the first one's, 16 bytes per lane. The vectors are
// declared 2-byte aligned: a rate field behind an odd number of 16-bit populations starts there,
// and the global memory instructions take any address (the whole field in 2-byte words instead
// made a 171 x 133 x 95 FP16 state 8 % slower to copy than the runtime's copy).
// Against the runtime's copies: 256^3 FP32 with its rate field 418 us (6.4 TB/s) and 518, 384^3
// FP16 735 us and 1044, 64^3 FP32 7.5 and 10.2.
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(2)));

struct CopyRange {
  const char* src;
  char* dst;
  size_t bytes;
};

template <bool CACHED>
__device__ __forceinline__ void copy_block(const CopyRange& r, size_t block) {
  const size_t at = (block * 256 + threadIdx.x) * 16;
  if (at + 16 <= r.bytes) {
    const v4f_any* from = reinterpret_cast<const v4f_any*>(r.src + at);
    v4f_any* to = reinterpret_cast<v4f_any*>(r.dst + at);
    if constexpr (CACHED) *to = *from;
    else __builtin_nontemporal_store(__builtin_nontemporal_load(from), to);
  } else {
    for (size_t b = at; b < r.bytes; b += 2)
      *reinterpret_cast<unsigned short*>(r.dst + b) = *reinterpret_cast<const unsigned short*>(r.src + b);
  }
}

template <bool CACHED>
__global__ __launch_bounds__(256) void copy_ranges_kernel(CopyRange a, CopyRange b, size_t blocks_a) {
  const size_t blk = blockIdx.x;
  if (blk < blocks_a) copy_block<CACHED>(a, blk);
  else copy_block<CACHED>(b, blk - blocks_a);
}

// Whether a kernel on `dev` may touch p: device memory of that device (anything else goes
// through the runtime's copy, which knows host and peer memory).
static bool local_memory(const void* p, int dev) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return at.type == hipMemoryTypeDevice && at.device == dev;
}

static hipError_t copy_by_runtime(const CopyRange& r, hipStream_t st) {
  return r.bytes ? hipMemcpyAsync(r.dst, r.src, r.bytes, hipMemcpyDeviceToDevice, st) : hipSuccess;
}

hipError_t launch_copy2(const void* src1, void* dst1, size_t bytes1, const void* src2, void* dst2, size_t bytes2,
                        hipStream_t st) {
  const CopyRange a{static_cast<const char*>(src1), static_cast<char*>(dst1), bytes1};
  const CopyRange b{static_cast<const char*>(src2), static_cast<char*>(dst2), bytes2};
  const size_t na = copy_blocks(bytes1), nb = copy_blocks(bytes2);
  hipDevice_t dev = 0;
  const auto halves = [](const CopyRange& r) {
    return ((reinterpret_cast<uintptr_t>(r.src) | reinterpret_cast<uintptr_t>(r.dst) | r.bytes) & 1) == 0;
  };
  const bool own = na + nb > 0 && copy_fits_launch(bytes1, bytes2) && halves(a) && halves(b) &&
                   hipStreamGetDevice(st, &dev) == hipSuccess && local_memory(src1, dev) && local_memory(dst1, dev) &&
                   (bytes2 == 0 || (local_memory(src2, dev) && local_memory(dst2, dev)));
  if (!own) {
    const hipError_t e = copy_by_runtime(a, st);
    return e == hipSuccess ? copy_by_runtime(b, st) : e;
  }
  // Source and destination within the 256 MB last-level cache: plain accesses and all the blocks
  // that fit (80 MB 25.6 us against 29.7 with nontemporal accesses, 5 blocks per CU; 127 MB 35.5
  // against 41); beyond it the streaming form of stream_copy_kernel (176 MB 53.5 against 56 us,
  // 670 MB 210 against 219).
  const dim3 grid(static_cast<unsigned>(na + nb));
  if (bytes1 + bytes2 <= (size_t(128) << 20))
    hipLaunchKernelGGL(copy_ranges_kernel<true>, grid, dim3(256), 0, st, a, b, na);
  else
    hipLaunchKernelGGL(copy_ranges_kernel<false>, grid, dim3(256), lds_cap_bytes(5, 0), st, a, b, na);
  return hipGetLastError();
}

}  // namespace lbm
