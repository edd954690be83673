// Paged K/V blocks in row layout ([block][KV head][16 slots][d], the layout a
// cache that stores each token's row contiguously uses) rewritten into the
// library's paged layouts, so a caller holding such a cache can run the
// decode step (App. E: the step attends over the cached rows of every
// stream; where a row lives is a storage choice).
//
//   K: [block][head][d/8][16][8], token t of a block in slot kslot(t) (bits
//      2 and 3 of t exchanged): 16-byte units of rows moved as they are
//   V: [block][head][d][16]: a 16 x d transpose per block and head through
//      LDS, 16-byte loads of rows, 16-byte stores of token runs
//
// A copy, bound by memory: every load and store is 16 bytes a lane.  One
// workgroup takes a (block, head) pair at a time (two where a pair is 128 units)
// with its K and V loads in flight together; the loads are non-temporal.  Measured on one
// MI355X, 16,384 blocks of 2 heads, d = 128, bf16 (537 MB read and written):
// two kernels that moved V two bytes at a time 153.6 us; this one 93.7 us (5.7
// TB/s), with 2 pairs in flight a workgroup 94.2, with 4 102.8 (107.5 with
// plain loads; no change with non-temporal stores).  The V rows are padded by 16 bytes in LDS: a
// store gathers one dim of 16 / sizeof(T) tokens, and the two halves of a
// dim's tokens (bf16) then lie in other banks.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

namespace padoc {
namespace {

constexpr int kSlots = 16;

// Buffers need only their element's alignment (the hardware takes 16-byte
// accesses at any address; aligned ones are as fast as if declared so).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <typename T>
struct Unit;
template <>
struct Unit<uint16_t> {
  typedef u32x4 type __attribute__((aligned(2)));
};
template <>
struct Unit<uint32_t> {
  typedef u32x4 type __attribute__((aligned(4)));
};

__device__ __forceinline__ int kslot(int t) { return (t & 3) | ((t & 4) << 1) | ((t & 8) >> 1); }

// T: uint16_t or uint32_t.  kUnits 16-byte units per pair and tensor, one or
// more per thread.
template <typename T, int D>
__global__ __launch_bounds__(256) void relayout_kv_kernel(const T* __restrict__ k_rows, const T* __restrict__ v_rows,
                                                          T* __restrict__ k_cache, T* __restrict__ v_cache,
                                                          int64_t n_pairs) {
  typedef typename Unit<T>::type unit_t;
  constexpr int E = 16 / (int)sizeof(T);       // elements per unit
  constexpr int UPR = D / E;                   // units per row
  constexpr int kUnits = kSlots * UPR;         // units per pair and tensor: 128 .. 512
  constexpr int kThreads = kUnits < 256 ? kUnits : 256;  // threads that share a pair
  constexpr int kShare = 256 / kThreads;       // pairs handled side by side
  constexpr int kPer = kUnits / kThreads;      // units per thread, tensor and pair
  constexpr int kRow = D + E;                  // padded LDS row
  __shared__ __attribute__((aligned(16))) T tile[kShare][kSlots * kRow];
  const int who = threadIdx.x / kThreads, u0 = threadIdx.x % kThreads;
  for (int64_t base = (int64_t)blockIdx.x * kShare; base < n_pairs; base += (int64_t)gridDim.x * kShare) {
    const int64_t pair = base + who;
    const bool on = pair < n_pairs;
    u32x4 kx[kPer], vx[kPer];
    if (on) {
      const unit_t* ks = reinterpret_cast<const unit_t*>(k_rows) + pair * kUnits;
      const unit_t* vs = reinterpret_cast<const unit_t*>(v_rows) + pair * kUnits;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        kx[i] = __builtin_nontemporal_load(ks + u0 + i * kThreads);
        vx[i] = __builtin_nontemporal_load(vs + u0 + i * kThreads);
      }
      unit_t* kd = reinterpret_cast<unit_t*>(k_cache) + pair * kUnits;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        // unit x of row t: dims E x .. of chunk (E x) / 8, at unit (E x % 8) / E of the piece
        const int unit = u0 + i * kThreads, t = unit / UPR, x = unit % UPR;
        constexpr int UPP = 8 / E;  // units per 8-dim piece
        kd[((x / UPP) * kSlots + kslot(t)) * UPP + x % UPP] = kx[i];
        *reinterpret_cast<u32x4*>(&tile[who][t * kRow + x * E]) = vx[i];
      }
    }
    __syncthreads();
    if (on) {
      unit_t* vd = reinterpret_cast<unit_t*>(v_cache) + pair * kUnits;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        // unit of the d-major block: dim, then E tokens
        constexpr int UPT = kSlots / E;
        const int unit = u0 + i * kThreads, dim = unit / UPT, t0 = (unit % UPT) * E;
        T y[E];
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = tile[who][(t0 + e) * kRow + dim];
        u32x4 o;
        if constexpr (sizeof(T) == 2)
          o = u32x4{y[0] | ((uint32_t)y[1] << 16), y[2] | ((uint32_t)y[3] << 16), y[4] | ((uint32_t)y[5] << 16),
                    y[6] | ((uint32_t)y[7] << 16)};
        else
          o = u32x4{y[0], y[1], y[2], y[3]};
        vd[unit] = o;
      }
    }
    __syncthreads();
  }
}

template <typename T, int D>
void launch(const void* k_rows, const void* v_rows, void* k_cache, void* v_cache, int64_t n_pairs, hipStream_t stream) {
  constexpr int per = std::max(1, 256 / (kSlots * D * (int)sizeof(T) / 16));
  const dim3 grid((unsigned)std::min<int64_t>((n_pairs + per - 1) / per, 1 << 20));
  hipLaunchKernelGGL((relayout_kv_kernel<T, D>), grid, dim3(256), 0, stream, static_cast<const T*>(k_rows),
                     static_cast<const T*>(v_rows), static_cast<T*>(k_cache), static_cast<T*>(v_cache), n_pairs);
}

}  // namespace

hipError_t launch_relayout_kv(const void* k_rows, const void* v_rows, void* k_cache, void* v_cache, int64_t n_blocks,
                              int Hkv, int D, int elem_bytes, hipStream_t stream) {
  if (n_blocks <= 0) return hipSuccess;
  const int64_t n_pairs = n_blocks * Hkv;
  if (elem_bytes == 2)
    D == 64 ? launch<uint16_t, 64>(k_rows, v_rows, k_cache, v_cache, n_pairs, stream)
            : launch<uint16_t, 128>(k_rows, v_rows, k_cache, v_cache, n_pairs, stream);
  else
    D == 64 ? launch<uint32_t, 64>(k_rows, v_rows, k_cache, v_cache, n_pairs, stream)
            : launch<uint32_t, 128>(k_rows, v_rows, k_cache, v_cache, n_pairs, stream);
  return hipGetLastError();
}

}  // namespace padoc
