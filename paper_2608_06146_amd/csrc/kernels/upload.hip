// Copy of a schedule from pinned host memory into the device workspace, ahead
// of the kernels that read it on the same stream.
//
// A kernel that reads the host memory over PCIe, not hipMemcpyAsync: above 16
// KB that call hands the copy to a DMA engine, and the hand-over in and out of
// the compute queue costs about 12 us, more than the copy.  Measured per
// (copy, small dependent kernel) pair on one MI355X, hipMemcpyAsync / this
// kernel: 16 KB 6.3 / 6.5 us, 32 KB 18.5 / 6.5, 128 KB 20.5 / 7.0, 512 KB
// 27.2 / 14.6, 2 MB 54.8 / 41.9, 8 MB 165 / 152.  64 workgroups keep enough
// reads in flight for the link (about 55 GB/s); 16 and 1024 were no faster at
// any size.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

namespace padoc {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void upload_kernel(u32x4* __restrict__ dst0, const u32x4* __restrict__ src0,
                                                     int64_t n0, u32x4* __restrict__ dst1,
                                                     const u32x4* __restrict__ src1, int64_t n1) {
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n0 + n1; i += step) {
    if (i < n0)
      dst0[i] = __builtin_nontemporal_load(src0 + i);
    else
      dst1[i - n0] = __builtin_nontemporal_load(src1 + (i - n0));
  }
}

}  // namespace

// One or two pieces, whole 16-byte units (the pinned copies and the workspace
// sections are padded to that); 16-byte aligned.
hipError_t launch_upload(void* dst0, const void* src0, size_t bytes0, void* dst1, const void* src1, size_t bytes1,
                         hipStream_t stream) {
  const int64_t n0 = (int64_t)((bytes0 + 15) / 16), n1 = (int64_t)((bytes1 + 15) / 16);
  if (n0 + n1 == 0) return hipSuccess;
  const dim3 grid((unsigned)std::min<int64_t>((n0 + n1 + 255) / 256, 64));
  hipLaunchKernelGGL(upload_kernel, grid, dim3(256), 0, stream, static_cast<u32x4*>(dst0),
                     static_cast<const u32x4*>(src0), n0, static_cast<u32x4*>(dst1), static_cast<const u32x4*>(src1),
                     n1);
  return hipGetLastError();
}

}  // namespace padoc
