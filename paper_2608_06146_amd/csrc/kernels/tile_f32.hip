// fp32 attention of a work item (packed forward and paged decode) on the
// matrix cores, v_mfma_f32_16x16x4_f32 (fp32 operands and accumulation).
// The schedules are the ones of the bf16 kernels.
//
// One workgroup per (work item, group of 16 columns; a column is a query
// token and one head of the item's KV head).  Its W wavefronts split the
// item's keys: wavefront w takes the 16-key blocks w, w+W, .. of the item's
// ranges in order, each straight from memory into matrix-core operand
// registers (K of the next block and V of this one are in flight while this
// block's scores are formed; no LDS stage, no barrier), keeps its own online
// softmax, and the W slices are merged through LDS at the end (App. E Attn
// equation, the softmax of disjoint key sets merged).
//
// What bounds it: at a few pages, a workgroup's chain of dependent loads
// (records, block ids, keys) and the merge; the products of the decode step
// below are about 6 us at the rate of a large fp32 product.  Hence the key
// split: a 448-key item of the small forward is 4 blocks a wavefront, not 7
// tiles one after the other.  W = 8 packed (few, long items).  W = 4 paged: 4
// wavefronts of 252 registers (64 of them accumulation registers; 256 is the
// most for this) leave a compute unit room for two workgroups,
// of which one waits for its first keys while the other computes (decode step
// of 4 pages of 1,152 shared keys and 16 branches, Hq 16, Hkv 2, d = 128,
// schedule resident: 37 us with 8, 31 with 4).  Without the K block in flight
// it was 32.
// Measured against one thread per column on the vector units (paged) and
// LDS-staged tiles with 8 interleaved key slices (packed), one MI355X, whole
// calls: that decode step 2,080 -> 48 us (33 since a kernel copies its
// schedule); packed forward of 256 + 64 + 4 x 32
// tokens, Hq 4, Hkv 1, d = 64: 31.8 -> 12.2 us (kernel 29 -> 9.4).
//
// Operand layout, lane (r, g) = (lane % 16, lane / 16), with every load one
// float4:
//   S^T = K Q^T     row r = key slot r of the block, contraction in the order
//                   the loads give: float4 j holds dims 16j+4g .. +3, so the
//                   product of (j, e) contracts dims 16j+4g+e, g = 0..3
//   O^T += V^T P^T  product i contracts the keys whose scores are element i
//                   of the four lane groups, so P^T is the score registers
//                   themselves.  Packed rows: float4 i of 64-dim group q is
//                   V[key 4g+i][64q+4r .. +3], so row r of block (q, c) is
//                   dim 64q+4r+c.  Paged (d-major) blocks: float4 of block db
//                   is V[dim 16db+r][4 tokens of the group].
// A wavefront's loads are whole 64-byte lines either way (paged: 1 KB
// contiguous).
#include <type_traits>

#include "device_common.hpp"

namespace padoc {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kCols = 16;   // columns per workgroup
constexpr int kKeys = 16;   // keys per block
constexpr int waves(bool paged) { return paged ? 4 : 8; }  // key slices
constexpr int kGroups = kTileCols / kCols;  // column groups of a full item

__device__ __forceinline__ f32x4_t load_f4(const float* p) { return *reinterpret_cast<const f32x4_t*>(p); }

template <int D, bool PAGED>
__global__ __launch_bounds__(64 * waves(PAGED)) void tile_f32_kernel(TileParams p, int n_full, int n_items) {
  constexpr int kWaves = waves(PAGED);
  constexpr int NJ = D / 16;  // float4 loads of a K or V block per lane
  // Workgroups of an item's column groups read the same keys: they are 8
  // apart, so that they run on one XCD (workgroup b on XCD b % 8) and share
  // its L2.  Items n_full .. n_items-1 have one column group.
  const int b = blockIdx.x;
  const int full_blocks = (n_full + 7) / 8 * 8 * kGroups;
  int item, cg;
  if (b < full_blocks) {
    item = (b / (8 * kGroups)) * 8 + b % 8;
    cg = (b / 8) % kGroups;
    if (item >= n_full) return;
  } else {
    item = n_full + b - full_blocks;
    cg = 0;
    if (item >= n_items) return;
  }
  const WorkRec w = load_scalar(&p.work[item]);
  if (cg * kCols >= w.ncol || w.rng_count <= 0) return;  // the whole workgroup
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int c = w.col0 + cg * kCols + r;
  const int t = c / p.G;
  const bool valid = cg * kCols + r < w.ncol && t < w.ntok;
  const int32_t qrow = valid ? p.toks[w.tok_begin + t] : 0;
  const int32_t hq = w.kvh * p.G + (c - t * p.G);
  const float* K = static_cast<const float*>(p.k);
  const float* V = static_cast<const float*>(p.v);
  const int64_t row_f = (int64_t)p.Hkv * D;  // floats of a packed K/V row
  // first key of this lane's 4 scores in a block (paged: slots 4g.. hold the
  // tokens of kslot)
  const int k0 = PAGED ? 4 * (((g & 1) << 1) | (g >> 1)) : 4 * g;

  f32x4_t q[NJ];
  {
    const float* qp = static_cast<const float*>(p.q) + ((int64_t)qrow * p.Hq + hq) * D + 4 * g;
#pragma unroll
    for (int j = 0; j < NJ; ++j) q[j] = valid ? load_f4(qp + 16 * j) : f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // Cursor over this wavefront's blocks.
  struct Cursor {
    int ri, blk;
    RangeRec R;
  };
  auto settle = [&](Cursor& x) -> bool {  // to a block that exists; false past the last
    while (x.blk * kKeys >= x.R.n_keys) {
      x.blk -= (x.R.n_keys + kKeys - 1) / kKeys;
      if (++x.ri >= w.rng_count) return false;
      x.R = load_scalar(&p.ranges[w.rng_begin + x.ri]);
    }
    return true;
  };
  auto limit_of = [&](const RangeRec& R) -> int {
    return !valid ? 0 : R.lim_off < 0 ? R.n_keys : p.lims[R.lim_off + t];
  };
  auto block_id = [&](const Cursor& x) -> int64_t {
    if constexpr (PAGED) return load_scalar(p.block_table + x.R.kv_start + x.blk);
    else return 0;
  };
  auto load_k = [&](const Cursor& x, int64_t id, f32x4_t (&kf)[NJ]) __attribute__((always_inline)) {
    if constexpr (PAGED) {
      const float* kp = K + (id * p.Hkv + w.kvh) * (int64_t)(D * kBlock) + (g >> 1) * (kBlock * 8) + r * 8 + 4 * (g & 1);
#pragma unroll
      for (int j = 0; j < NJ; ++j) kf[j] = load_f4(kp + j * (2 * kBlock * 8));
    } else {
      const int key = min(x.blk * kKeys + r, x.R.n_keys - 1);  // past the end: the last row, masked
      const float* kp = K + (x.R.kv_start + key) * row_f + w.kvh * D + 4 * g;
#pragma unroll
      for (int j = 0; j < NJ; ++j) kf[j] = load_f4(kp + 16 * j);
    }
  };
  // Packed: vf[4q+i]; paged: vf[db].
  auto load_v = [&](const Cursor& x, int64_t id, f32x4_t (&vf)[NJ]) __attribute__((always_inline)) {
    if constexpr (PAGED) {
      const float* vp = V + (id * p.Hkv + w.kvh) * (int64_t)(D * kBlock) + r * kBlock + k0;
#pragma unroll
      for (int db = 0; db < NJ; ++db) vf[db] = load_f4(vp + db * 16 * kBlock);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = min(x.blk * kKeys + k0 + i, x.R.n_keys - 1);
        const float* vp = V + (x.R.kv_start + key) * row_f + w.kvh * D + 4 * r;
#pragma unroll
        for (int qd = 0; qd < D / 64; ++qd) vf[4 * qd + i] = load_f4(vp + 64 * qd);
      }
    }
  };

  float m = -INFINITY, l = 0.f;  // l: this lane's scores only, until the merge
  f32x4_t acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const float sl2 = p.scale_log2;

  Cursor C{0, wave, load_scalar(&p.ranges[w.rng_begin])};
  bool go = settle(C);
  if (go) {
    f32x4_t kf[2][NJ], vf[NJ];
    int lim = limit_of(C.R);
    int64_t id = block_id(C);
    load_k(C, id, kf[0]);
    auto step = [&](auto xc) __attribute__((always_inline)) {
      constexpr int X = decltype(xc)::value;
      // The next block (this one again past the last: every step issues the
      // same loads, so waits stay exact).
      Cursor N = C;
      N.blk += kWaves;
      const bool more = settle(N);
      if (!more) N = C;
      const int lim_n = N.ri != C.ri ? limit_of(N.R) : lim;
      const int64_t id_n = block_id(N);
      load_v(C, id, vf);
      // Four sums of D/4 products each: shorter chains of roundings, and
      // products that do not wait for one another.
      f32x4_t Sp[4];
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          Sp[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[X][j][e], q[j][e], j ? Sp[e] : f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      f32x4_t S = (Sp[0] + Sp[1]) + (Sp[2] + Sp[3]);
      load_k(N, id_n, kf[X ^ 1]);
      const int kb = C.blk * kKeys;
      const bool partial = kb + kKeys > C.R.min_lim;
      // Masked without a branch: the compiler leaves out the wait states
      // between a matrix product and a read of its result where the read is
      // the target of a branch around a longer block.
      const int seen = partial ? lim - kb - k0 : 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) S[i] = i < seen ? S[i] : -INFINITY;
      float mx = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3]));
      mx = max_lane_halves(max_lane_rows(mx)) * sl2;
      if (__any(mx > m)) {
        const float mn = fmaxf(m, mx);
        const float alpha = mn == -INFINITY ? 1.f : fast_exp2(m - mn);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[j] *= alpha;
      }
      const float ms = m == -INFINITY ? 0.f : m;
      float e[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        e[i] = fast_exp2(fmaf(S[i], sl2, -ms));
        l += e[i];
      }
      bool plain = true;
      if (PAGED && partial) {
        // Some column of the block does not see some of its slots, which may
        // hold anything; 0 * inf would be NaN.  Slots past the range's end
        // are zeroed; a non-finite value in a slot that only some columns
        // see goes the slow way below.
        bool odd = false;
#pragma unroll
        for (int db = 0; db < NJ; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (kb + k0 + i >= C.R.n_keys) vf[db][i] = 0.f;
            odd |= !(fabsf(vf[db][i]) < INFINITY);
          }
        plain = !__any(odd);
      }
      if (plain) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(PAGED ? vf[j][i] : vf[4 * (j / 4) + i][j % 4], e[i], acc[j], 0, 0, 0);
      } else {
        for (int k = 0; k < kKeys && kb + k < C.R.n_keys; ++k) {
          // token k's probability for this column: element k % 4 of the lane
          // group whose tokens start at k - k % 4
          const int gk = (((k >> 2) & 1) << 1) | (k >> 3);
          const float ek = __shfl(k % 4 == 0 ? e[0] : k % 4 == 1 ? e[1] : k % 4 == 2 ? e[2] : e[3], r + 16 * gk);
          if (kb + k >= lim) continue;
          const float* vp = V + (id * p.Hkv + w.kvh) * (int64_t)(D * kBlock) + 4 * g * kBlock + k;
#pragma unroll
          for (int db = 0; db < NJ; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[db][i] = fmaf(ek, vp[(16 * db + i) * kBlock], acc[db][i]);
        }
      }
      C = N;
      lim = lim_n;
      id = id_n;
      go = more;
    };
    for (;;) {
      step(std::integral_constant<int, 0>{});
      if (!go) break;
      step(std::integral_constant<int, 1>{});
      if (!go) break;
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  // Merge: every wavefront writes its slice, then wavefront v sums float4 v
  // of all slices.  Float4 v of lane (r, g): packed, v = 4q+i: dims
  // 64q+16g+4i .. +3; paged, dims 16v+4g .. +3.
  __shared__ f32x4_t So[kWaves][NJ][64];
  __shared__ float2 Sml[kWaves][kCols];
  if (g == 0) Sml[wave][r] = make_float2(m, l);
#pragma unroll
  for (int v = 0; v < NJ; ++v) {
    if constexpr (PAGED) {
      So[wave][v][lane] = acc[v];
    } else {
      const int qd = v / 4, i = v % 4;
      So[wave][v][lane] = f32x4_t{acc[4 * qd][i], acc[4 * qd + 1][i], acc[4 * qd + 2][i], acc[4 * qd + 3][i]};
    }
  }
  __syncthreads();
  if (!valid) return;
  float M = -INFINITY;
  float2 ml[kWaves];
#pragma unroll
  for (int s = 0; s < kWaves; ++s) {
    ml[s] = Sml[s][r];
    M = fmaxf(M, ml[s].x);
  }
  const float Ms = M == -INFINITY ? 0.f : M;
  float L = 0.f;
#pragma unroll
  for (int s = 0; s < kWaves; ++s) {
    ml[s].x = fast_exp2(ml[s].x - Ms);
    L = fmaf(ml[s].y, ml[s].x, L);
  }
#pragma unroll
  for (int v = wave; v < NJ; v += kWaves) {
    f32x4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kWaves; ++s) o += So[s][v][lane] * ml[s].x;
    const int d0 = PAGED ? 16 * v + 4 * g : 64 * (v / 4) + 16 * g + 4 * (v % 4);
    if constexpr (PAGED)
      *reinterpret_cast<f32x4_t*>(p.part_o + ((int64_t)w.out_base + c) * D + d0) = o;
    else
      *reinterpret_cast<f32x4_t*>(static_cast<float*>(p.o) + ((int64_t)qrow * p.Hq + hq) * D + d0) = o * (1.f / L);
  }
  if (wave != 0 || g != 0) return;
  if constexpr (PAGED) {
    const int64_t slot = (int64_t)w.out_base + c;
    p.part_ml[2 * slot] = M;
    p.part_ml[2 * slot + 1] = L;
  } else {
    p.lse[(int64_t)qrow * p.Hq + hq] = (M + __log2f(L)) * kLn2;
  }
}

}  // namespace

// n_full: the first items of the schedule, of up to kTileCols columns each
// (every packed item; the shared items of a decode step); the others are
// private decode items of one column group.
hipError_t launch_tile_f32(const TileParams& p, int n_full, int n_items, int D, bool paged, hipStream_t stream) {
  static_assert(kCols == kPrivateCols, "a private item is one column group");
  if (n_items <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n_full + 7) / 8 * 8 * kGroups + (n_items - n_full))), block(64 * waves(paged));
  if (paged) {
    if (D == 64)
      hipLaunchKernelGGL((tile_f32_kernel<64, true>), grid, block, 0, stream, p, n_full, n_items);
    else
      hipLaunchKernelGGL((tile_f32_kernel<128, true>), grid, block, 0, stream, p, n_full, n_items);
  } else {
    if (D == 64)
      hipLaunchKernelGGL((tile_f32_kernel<64, false>), grid, block, 0, stream, p, n_full, n_items);
    else
      hipLaunchKernelGGL((tile_f32_kernel<128, false>), grid, block, 0, stream, p, n_full, n_items);
  }
  return hipGetLastError();
}

}  // namespace padoc
