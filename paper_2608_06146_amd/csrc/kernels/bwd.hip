// Backward of the packed tree forward (bf16, gfx950 matrix cores).
//
// The gradient of sum(dO * O) with O = softmax(scale * q K^T + A_M) V over
// each query's visible keys (App. E Attn equation with the ancestor mask;
// App. C tree-varlen relation, the backend the paper trains with), written
// per query row i and visible key j:
//   P_ij  = exp(scale q_i.k_j - LSE_i)      (recomputed from the forward LSE)
//   dV_j  = sum_i P_ij dO_i
//   dP_ij = dO_i . v_j,   D_i = dO_i . O_i
//   dS_ij = P_ij (dP_ij - D_i)
//   dQ_i  = scale sum_j dS_ij k_j,   dK_j = scale sum_i dS_ij q_i
// Four kernels:
//   bwd_tokens  the key-major items' token lists, from their compact form
//   bwd_dq      query-major: the forward's work items (256 columns x the
//               item's key ranges); per 64-key tile S^T, dP^T, dS^T and
//               dQ^T += K^T dS^T; dQ is complete per item and written directly.
//               Its columns' D and LSE are kept for bwd_dkdv.
//   bwd_dkdv    key-major: up to 128 keys of one segment against the query
//               columns that see them, 64 columns per step; every wavefront
//               holds dK and dV of 32 keys and takes 32 of the step's columns
//   bwd_reduce  sums of the pieces of split key runs -> bf16 dK, dV (round to
//               nearest even); zero rows where no query sees a key
// All products are v_mfma_f32_32x32x16_bf16 with fp32 accumulation.  An
// operand whose contraction index is not contiguous in memory (K^T for dQ,
// dO^T and Q^T for dV and dK) is read from its row-major LDS block with the
// transposing LDS read of gfx950 (within each group of 16 lanes, lane r
// supplies the address of 4 consecutive elements and lane 4a+b receives
// element b of the pieces of lanes a, 4+a, 8+a and 12+a), two reads per
// operand, in the key / column order of the probabilities' registers.
#include <stddef.h>

#include <algorithm>

#include "device_common.hpp"
#include "fwd_item.hpp"

namespace padoc {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kThreads = 512;
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ bf16x8_t as_bf16x8(const uint4& u) { return *reinterpret_cast<const bf16x8_t*>(&u); }

// Row-major LDS blocks of CPR 16-byte chunks per row store chunk c of row r
// at chunk c ^ sw(r): the row reads of the matrix products (16 rows, one
// chunk) and the transposing reads (4 rows, 4 aligned chunks) then each
// touch distinct banks.  CPR = 16 (d = 128): one row per 256-byte bank row;
// CPR = 8 (d = 64): two rows per bank row, so the swizzle keys on the row
// pair.
template <int CPR>
__device__ __forceinline__ int swizzled_chunk(int r, int c) {
  const int sw = CPR == 16 ? (((r & 3) << 2) | ((r >> 2) & 3)) : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
  return c ^ sw;
}

// ------------------------------------------------------------------ token lists

// The key-major items' token lists (query row and limit per token) from their
// compact form, one wavefront per piece: the lists of the 8-page sample are
// 6 MB, 100 us over the bus, their pieces 0.2 MB.
__global__ __launch_bounds__(256) void bwd_tokens_kernel(BwdParams p) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= p.n_btokens) return;
  const BwdTokens k = load_scalar(p.btokens + i);
  for (int j = lane; j < k.count; j += 64) {
    p.btoks[(int64_t)k.dst + j] = k.row0 + j;
    p.blims[(int64_t)k.dst + j] = min(k.lim0 + k.slope * j, k.lim_max);
  }
}

// ------------------------------------------------------------------ dQ

// 8 wavefronts of 32 columns.  A wavefront takes a 64-key tile in two halves:
// the products of one run beside the vector work of the other.  K and V come
// by direct global -> LDS loads two tiles ahead, into three stages, one barrier
// a tile; no step waits for more than its own tile (with waits for every load
// in flight in each step, the backward of 8 ragged pages took 3,376 us instead
// of 3,274, of one page 212.5 instead of 209.2).
template <int D>
__global__ __launch_bounds__(kThreads) void bwd_dq_kernel(BwdParams p) {
  constexpr int KT = kTileKeys;  // 64 keys per tile
  constexpr int NKK = D / 16;
  constexpr int NDB = D / 32;
  constexpr int CPR = D / 8;              // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;           // rows per 1 KB load
  constexpr int IPW = KT / RPI / 8;       // 1 KB loads per wavefront, tile and tensor
  constexpr int kStages = 3, kTile = KT * D;
  // K and V stages: KT rows of D elements with swizzled 16-byte chunks, read
  // by rows for S and dP and transposed (K^T) for dQ.
  __shared__ __attribute__((aligned(1024))) uint16_t sm[kStages][2][kTile];
  auto at = [&](int r, int c) { return r * D + (swizzled_chunk<CPR>(r, c) << 3); };

  const WorkRec w = load_scalar(&p.work[blockIdx.x]);
  if (w.rng_count <= 0) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int G = p.G, kvh = w.kvh;

  const int col = wave * 32 + l32;
  const int tok = col / G;
  const bool valid = tok < w.ntok;
  const int32_t qrow = valid ? p.toks[w.tok_begin + tok] : 0;
  const int64_t row = (int64_t)qrow * p.Hq + kvh * G + (valid ? col - tok * G : 0);
  bf16x8_t bq[NKK], bdo[NKK];
  float lse2, dcol;
  {
    const uint16_t* qp = static_cast<const uint16_t*>(p.q) + row * D + hf * 8;
    const uint16_t* gp = static_cast<const uint16_t*>(p.dout) + row * D + hf * 8;
    const uint16_t* op = static_cast<const uint16_t*>(p.o) + row * D + hf * 8;
    // D = dO . O (a lane half holds half of the dims), kept for the key-major
    // kernel with -LSE / scale
    float dd = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      bq[kk] = as_bf16x8(valid ? load16(qp + kk * 16) : make_uint4(0, 0, 0, 0));
      bdo[kk] = as_bf16x8(valid ? load16(gp + kk * 16) : make_uint4(0, 0, 0, 0));
      const uint4 o4 = valid ? load16(op + kk * 16) : make_uint4(0, 0, 0, 0);
      const uint32_t ow[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dd = fmaf(__uint_as_float(ow[i] << 16), (float)bdo[kk][2 * i], dd);
        dd = fmaf(__uint_as_float(ow[i] & 0xffff0000u), (float)bdo[kk][2 * i + 1], dd);
      }
    }
    dcol = dd + __shfl_xor(dd, 32);
    const float lse = valid ? p.lse[row] : 0.f;
    lse2 = lse * kLog2e;
    if (valid && hf == 0) {
      p.nd[row] = -dcol;
      p.nl[row] = -lse / p.scale_kv;
    }
  }
  const float sl2 = p.scale_log2;

  int n_tiles = 0;
  for (int r = 0; r < w.rng_count; ++r)
    n_tiles += (load_scalar(&p.ranges[w.rng_begin + r]).n_keys + KT - 1) / KT;
  struct Cursor {
    int ri, kt;
    RangeRec R;
  };
  auto advance = [&](Cursor& c) {  // past the last tile it stays on a valid one
    if (++c.kt * KT >= c.R.n_keys) {
      c.kt = 0;
      if (++c.ri < w.rng_count) c.R = load_scalar(&p.ranges[w.rng_begin + c.ri]);
    }
  };
  // This wavefront's loads of the tile at cursor c into stage s.  Rows past
  // the range's end repeat its last row (finite values whose scores the mask
  // removes).
  const uint32_t HD = (uint32_t)p.Hkv * D;
  const int ld_r = wave * IPW * RPI + lane / CPR;
  auto load = [&](const Cursor& c, int s) __attribute__((always_inline)) {
    const int kbase = c.kt * KT, last = c.R.n_keys - 1 - kbase;
    const int64_t first = tile::uniform64(c.R.kv_start + kbase) * (int64_t)HD;
    const uint16_t* kp = static_cast<const uint16_t*>(p.k) + first;
    const uint16_t* vp = static_cast<const uint16_t*>(p.v) + first;
    const uint32_t sk = tile::lds_addr(sm[s][0]) + wave * IPW * 1024, sv = tile::lds_addr(sm[s][1]) + wave * IPW * 1024;
#pragma unroll
    for (int j = 0; j < IPW; ++j) {
      const int r = ld_r + j * RPI;
      const uint32_t off = 2 * (__umul24((uint32_t)min(r, last), HD) + (uint32_t)kvh * D + 8 * swizzled_chunk<CPR>(r, lane % CPR));
      tile::dma16(kp, off, sk + j * 1024);
      tile::dma16(vp, off, sv + j * 1024);
    }
  };
  auto lim_of = [&](const RangeRec& R) -> int {
    return R.lim_off < 0 ? R.n_keys : (valid ? p.lims[R.lim_off + tok] : 0);
  };
  // A limit is waited for before the step that uses it: pending at a loop's
  // back edge, the compiler, which does not count the loads to LDS, could only
  // wait for every load in flight in each step.
  auto settle = [&](int& x) __attribute__((always_inline)) { asm volatile("" : "+v"(x)); };

  // Fragment addresses (bytes): rows of K or V: row mb*32 + l32, d = kk*16 +
  // hf*8 ..; K^T (d on M, keys on K) for keys mb*32 + 16j + 4*half + {0..3},
  // {8..11} of d block db: two transposing reads (lane r of a 16-lane group
  // supplies key row .. + r/4, elements d0 + 4*(r%4) .. +3).
  typedef __attribute__((address_space(3))) const bf16x8_t lds_frag;
  const int tr_r = 4 * hf + ((lane & 15) >> 2), tr_c = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
  const uint32_t a_row = 2 * at(l32, hf), a_tr = 2 * (at(tr_r, tr_c) + 4 * (lane & 1));
  const uint32_t lds0 = tile::lds_addr(sm);
  constexpr uint32_t kV = 2 * kTile;  // V tile after the K tile of a stage
  // A base that the compiler takes for a new value: the block addresses are
  // formed for each product group (one operation each), not kept.
  auto base = [&](uint32_t st, uint32_t a) __attribute__((always_inline)) -> uint32_t {
    uint32_t x = st + a;
    asm volatile("" : "+v"(x));
    return x;
  };
  auto ktf = [&](uint32_t b, int mb, int j, int db) __attribute__((always_inline)) -> bf16x8_t {
    const uint32_t to = mb * 64 * D + j * 32 * D;
    return tile::tr_pair_at((b ^ (uint32_t)(db << 6)) + to, (b ^ (uint32_t)((db << 6) | 32)) + to + 16 * D);
  };

  f32x16_t acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;
  // One tile, in stage st: S and dP of half 0; those of half 1 beside the dS
  // of half 0; dQ of half 0 beside the dS of half 1; dQ of half 1.  Element i
  // of half mb is key mb*32 + (i/4)*8 + hf*4 + i%4 of the tile, visible below
  // rel (relative to the tile and the lane half).
  auto tile_step = [&](uint32_t st, bool partial, int rel) __attribute__((always_inline)) {
    constexpr int kPre = 4, NA = 2 * NKK, NQ = 2 * NDB;
    f32x16_t S[2], dP[2];
    bf16x8_t ds[2][2];
    float x[8];
    // S and dP products of half mb, hook(i) after product i
    auto scores = [&](auto mbc, auto&& hook) __attribute__((always_inline)) {
      constexpr int mb = decltype(mbc)::value;
      const uint32_t b = base(st, a_row);
      auto frag = [&](int i) __attribute__((always_inline)) -> bf16x8_t {
        return *(lds_frag*)(uintptr_t)((b ^ (uint32_t)((i >> 1) << 5)) + (i & 1 ? kV : 0) + mb * 64 * D);
      };
      bf16x8_t f[kPre];
#pragma unroll
      for (int i = 0; i < kPre; ++i) f[i] = frag(i);
      __builtin_amdgcn_sched_barrier(0);
      tile::static_for<NA>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, kk = i >> 1;
        if constexpr (i & 1)
          dP[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kPre], bdo[kk], kk ? dP[mb] : f32x16_t{}, 0, 0, 0);
        else
          S[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kPre], bq[kk], kk ? S[mb] : f32x16_t{}, 0, 0, 0);
        if constexpr (i + kPre < NA) f[i % kPre] = frag(i + kPre);
        hook(ic);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    auto dq_half = [&](auto mbc, auto&& hook) __attribute__((always_inline)) {
      constexpr int mb = decltype(mbc)::value;
      const uint32_t b = base(st, a_tr);
      bf16x8_t f[kPre];
#pragma unroll
      for (int i = 0; i < kPre; ++i) f[i] = ktf(b, mb, i / NDB, i % NDB);
      __builtin_amdgcn_sched_barrier(0);
      tile::static_for<NQ>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, j = i / NDB, db = i % NDB;
        acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[i % kPre], ds[mb][j], acc[db], 0, 0, 0);
        if constexpr (i + kPre < NQ) f[i % kPre] = ktf(b, mb, (i + kPre) / NDB, (i + kPre) % NDB);
        hook(ic);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    auto mask = [&](auto mbc) __attribute__((always_inline)) {
      constexpr int mb = decltype(mbc)::value;
      if (partial) {
#pragma unroll
        for (int i = 0; i < 16; ++i) S[mb][i] = mb * 32 + (i >> 2) * 8 + (i & 3) < rel ? S[mb][i] : -INFINITY;
      }
    };
    // dS of half mb in the slots after products 2 .. N-1 of another group
    // (its last score product has landed by then)
    auto finish = [&](auto mbc, auto nc, auto ic) __attribute__((always_inline)) {
      constexpr int mb = decltype(mbc)::value, n = decltype(nc)::value - 2, k = decltype(ic)::value - 2;
      if constexpr (k == 0) mask(mbc);
      if constexpr (k >= 0)
        tile::static_for<16 * (k + 1) / n - 16 * k / n>([&](auto uc) __attribute__((always_inline)) {
          constexpr int i = 16 * k / n + decltype(uc)::value;
          const float pr = fast_exp2(fmaf(S[mb][i], sl2, -lse2));
          x[i % 8] = pr * (dP[mb][i] - dcol);
          if constexpr (i % 8 == 7) {
#pragma unroll
            for (int e = 0; e < 8; ++e) ds[mb][i / 8][e] = (__bf16)x[e];
          }
        });
    };
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;
    scores(H0{}, [&](auto) {});
    scores(H1{}, [&](auto ic) __attribute__((always_inline)) { finish(H0{}, std::integral_constant<int, NA>{}, ic); });
    dq_half(H0{}, [&](auto ic) __attribute__((always_inline)) { finish(H1{}, std::integral_constant<int, NQ>{}, ic); });
    dq_half(H1{}, [&](auto) {});
  };

  // Step t computes stage t % 3; the loads of tile t+2 go to the stage of tile
  // t-1, which every wavefront has read before this step's barrier, and each
  // wavefront waits for its own loads of tile t before it (only those of tile
  // t+1 may still be in flight).  Past the item's last tile the cursor stays
  // on a valid one.
  Cursor C{0, 0, load_scalar(&p.ranges[w.rng_begin])}, L = C;
  int lim = lim_of(C.R);
  load(L, 0);
  advance(L);
  load(L, 1);
  advance(L);
  int s = 0;
  if (wave * 32 >= w.ntok * G) {
    // No column of this wavefront is in use (half an item): its part of the
    // loads and barriers, the SIMD left to the wavefront that shares it.
    for (int t = 0; t < n_tiles; ++t) {
      tile::wait_vm<2 * IPW>();
      tile::bar();
      load(L, s == 0 ? 2 : s - 1);
      advance(L);
      s = s == 2 ? 0 : s + 1;
    }
    __builtin_amdgcn_s_waitcnt(0);
    return;
  }
  settle(lim);
  for (int t = 0; t < n_tiles; ++t) {
    tile::wait_vm<2 * IPW>();
    tile::bar();
    load(L, s == 0 ? 2 : s - 1);
    advance(L);
    const int kb = C.kt * KT;
    tile_step(lds0 + s * (4 * kTile), kb + KT > C.R.min_lim, lim - kb - hf * 4);
    const int ri = C.ri;
    advance(C);
    if (C.ri != ri && t + 1 < n_tiles) {
      lim = lim_of(C.R);
      settle(lim);
    }
    s = s == 2 ? 0 : s + 1;
  }
  __builtin_amdgcn_s_waitcnt(0);

  if (!valid) return;
  const float sc = p.scale;
  uint16_t* op = static_cast<uint16_t*>(p.dq) + row * D;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x16_t& v = acc[db];
      uint2 pk;
      pk.x = (uint32_t)f32_to_bf16_bits(v[4 * i4] * sc) | ((uint32_t)f32_to_bf16_bits(v[4 * i4 + 1] * sc) << 16);
      pk.y = (uint32_t)f32_to_bf16_bits(v[4 * i4 + 2] * sc) | ((uint32_t)f32_to_bf16_bits(v[4 * i4 + 3] * sc) << 16);
      *reinterpret_cast<uint2*>(op + db * 32 + i4 * 8 + hf * 4) = pk;
    }
}

// ------------------------------------------------------------------ dK, dV

// 8 wavefronts, 4 groups of 32 keys by 2 halves of a step's 64 columns: each
// forms S, P, dP and dS of its 32 x 32 block and adds its dV and dK, so that
// no block value crosses wavefronts and a step needs one barrier; the two
// column halves of a key group add up through LDS at the end.  Q and dO rows
// come by direct global -> LDS loads, two steps ahead, into three stages.
// Accumulators start at -LSE / scale and -D, which saves a subtraction each.
//
// What bounds it: a step's 32 products per wavefront are 2,048 cycles of each
// matrix core (two wavefronts a SIMD), its fragment reads 288 KB of LDS, about
// 2,500 cycles; it takes about 4,000.  More columns or keys per fragment read
// would need more registers than two wavefronts a SIMD have (this one takes
// 252, with a quarter of K in LDS).  Measured on one MI355X (d = 128, Hq 16,
// Hkv 2), against wavefront pairs that passed P through LDS inside each
// 32-column block: 8 ragged pages (43k tokens) 2,997 -> 1,870 us, one page of
// 3,400 tokens 399 -> 118 us.  Of the latter, the sums of split runs: added
// with fp32 atomics 336 us, through slots 118 + 8.6 for the reduction (atomics
// on 194 pieces ran at about 45 G/s).
// WIDE: Q or the list of limits is 4 GB or more, so places in them need 64 bits.
template <int D, bool WIDE>
__global__ __launch_bounds__(kThreads) void bwd_dkdv_kernel(BwdParams p) {
  constexpr int NKK = D / 16;
  constexpr int NDB = D / 32;
  constexpr int CPR = D / 8;            // 16-byte chunks per row
  constexpr int COLS = 64;              // columns per step
  constexpr int RPI = 64 / CPR;         // rows per 1 KB load
  constexpr int IPW = COLS / RPI / 8;   // 1 KB loads per wavefront, step and tensor
  constexpr int kStages = 3;
  struct Stage {
    uint16_t q[COLS * D];  // Q rows (row = column of the step), swizzled chunks
    uint16_t g[COLS * D];  // dO rows
    float nl[COLS];        // -LSE / scale per column
    float nd[COLS];        // -dO . O per column
    int lm[COLS];          // keys of the item the column sees
  };
  // the stages; at the end, the exchange of the column halves' sums
  constexpr int kExchange = 2 * 4 * 2 * 64 * (int)sizeof(f32x16_t);
  constexpr int kStageBytes = kStages * (int)sizeof(Stage);
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kStageBytes > kExchange ? kStageBytes : kExchange];
  Stage* st = reinterpret_cast<Stage*>(smem);
  struct Columns {
    uint32_t row[COLS];  // query row * Hq + head   (these three in bytes from
    uint32_t val[COLS];  // the same                 the start of the array they
    uint32_t lim[COLS];  // index of the limit       index, unless WIDE)
  };
  __shared__ Columns cols[4];  // of step t in list t % 4
  auto at = [&](int r, int c) { return r * D + (swizzled_chunk<CPR>(r, c) << 3); };
  // The lane index as a value the compiler takes for a new one: what each step
  // derives from it (addresses) is formed in the step, a few operations, and
  // holds no register through the products.
  auto fresh_lane = [&]() __attribute__((always_inline)) -> int {
    int x = threadIdx.x & 63;
    asm volatile("" : "+v"(x));
    return x;
  };

  const BwdRec b = load_scalar(&p.bwd[blockIdx.x]);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int kg = wave & 3, cb = wave >> 2;  // this wavefront's 32 keys and 32 columns of a step
  const int key = kg * 32 + l32, key_hi = kg * 32 + 32;
  const bool idle = kg * 32 >= b.n_keys;  // no key: stages and barriers only
  const int G = p.G, kvh = b.kvh;
  const int64_t Hkv = p.Hkv;
  const int c_begin = b.col0, c_end = b.col0 + b.ncol;

  // B operands of S = Q K^T and dP = dO V^T: this lane's key, d = kk*16 + hf*8 ..
  // At d = 128 the last kKL pieces of K wait in LDS (both column halves of a
  // key group read the same), else the sums would not all fit the registers.
  constexpr int kKL = D == 128 ? 4 : 0, NKR = NKK - kKL;
  __shared__ __attribute__((aligned(16))) bf16x8_t Kl[4][kKL > 0 ? kKL : 1][64];
  bf16x8_t bk[NKR], bv[NKK];
  {
    const int kc = key < b.n_keys ? key : b.n_keys - 1;
    const int64_t off = ((b.key_row0 + kc) * Hkv + kvh) * D + hf * 8;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      bv[kk] = as_bf16x8(load16(static_cast<const uint16_t*>(p.v) + off + kk * 16));
      const bf16x8_t x = as_bf16x8(load16(static_cast<const uint16_t*>(p.k) + off + kk * 16));
      if (kk < NKR)
        bk[kk] = x;
      else if (cb == 0)
        Kl[kg][kk - NKR][lane] = x;
    }
  }

  // Staging.  1 KB load i = wave*IPW + j of a tensor fills rows RPI*i ..
  // RPI*i+RPI-1 of a stage; lane l fetches the chunk of row RPI*i + l/CPR whose
  // place is l%CPR.  Row r of the step starting at column c is column c + r
  // of the item: token (c + r) / G, head (c + r) % G.  One wavefront (7) works
  // the columns out, a step before the others read them from LDS: c's own
  // token and head advance in scalar registers, the quotient of the small
  // rest is a multiplication (exact: x < 128, G <= 64).  Columns past c_end
  // repeat the last one, whose Q, dO, LSE and D are finite, and count as
  // seeing no key.
  const int t_end = (c_end - 1) / G, h_end = (c_end - 1) % G;
  const uint32_t inv_g = 65536u / (uint32_t)G + 1;
  const int t64 = COLS / G, h64 = COLS % G;
  int f_c = c_begin, f_t = c_begin / G, f_h = c_begin % G;  // next step to list
  int l_c = f_c, l_t = f_t, l_h = f_h;              // the step fetched last
  auto column = [&](int c, int t0, int h0, int& t, int& h) __attribute__((always_inline)) {
    const uint32_t x = (uint32_t)(h0 + lane);
    const uint32_t dt = (x * inv_g) >> 16;
    const bool ok = c + lane < c_end;
    t = ok ? t0 + (int)dt : t_end;
    h = ok ? (int)(x - dt * (uint32_t)G) : h_end;
  };
  // The query rows of the next columns into list u, by a load to LDS like the
  // others: the compiler would wait for one into a register, and with it for
  // every load in flight, in each step.
  auto fetch_rows = [&](int u) __attribute__((always_inline)) {
    int t, h;
    column(f_c, f_t, f_h, t, h);
    if constexpr (WIDE)
      tile::dma4_v(p.btoks + b.tok_begin + t, tile::lds_addr(cols[u].row));
    else
      tile::dma4(p.btoks, 4 * (uint32_t)(b.tok_begin + t), tile::lds_addr(cols[u].row));
    l_c = f_c, l_t = f_t, l_h = f_h;
    f_c += COLS;
    f_t += t64;
    f_h += h64;
    if (f_h >= G) {
      f_h -= G;
      ++f_t;
    }
  };
  auto list_rows = [&](int u) __attribute__((always_inline)) {  // the columns fetched last, list u, from their query rows
    int t, h;
    column(l_c, l_t, l_h, t, h);
    const uint32_t row = cols[u].row[lane] * (uint32_t)p.Hq + (uint32_t)(kvh * G + h);
    cols[u].row[lane] = WIDE ? row : row * (2 * D);
    cols[u].val[lane] = WIDE ? row : row * 4;
    cols[u].lim[lane] = WIDE ? (uint32_t)(b.lim_begin + t) : 4 * (uint32_t)(b.lim_begin + t);
  };
  // Loads of the columns of list u into stage s: 2*IPW loads of 1 KB and one
  // of 256 bytes per wavefront (wavefronts 3-7 repeat wavefront 2's).
  auto load = [&](int u, int s) __attribute__((always_inline)) {
    const int ln = fresh_lane();
    const uint32_t r_off = wave * IPW * RPI + ln / CPR;
    const uint32_t c_off = 16 * swizzled_chunk<CPR>(r_off, ln % CPR);
    const uint32_t sq = tile::lds_addr(st[s].q) + wave * IPW * 1024, sg = tile::lds_addr(st[s].g) + wave * IPW * 1024;
#pragma unroll
    for (int j = 0; j < IPW; ++j) {
      // the row of load 1 is 4 further on: its swizzle differs in bit 0
      static_assert(IPW == 1 || (IPW == 2 && CPR == 16), "chunk of load 1");
      const uint32_t row = cols[u].row[r_off + j * RPI];
      const uint32_t c = c_off ^ (16 * j);
      if constexpr (WIDE) {
        const uint64_t off = (uint64_t)row * (2 * D) + c;
        tile::dma16_v(static_cast<const char*>(p.q) + off, sq + j * 1024);
        tile::dma16_v(static_cast<const char*>(p.dout) + off, sg + j * 1024);
      } else {
        tile::dma16(p.q, row + c, sq + j * 1024);
        tile::dma16(p.dout, row + c, sg + j * 1024);
      }
    }
    const void* base = wave == 0 ? (const void*)p.nl : wave == 1 ? (const void*)p.nd : (const void*)p.blims;
    const uint32_t val = wave < 2 ? cols[u].val[ln] : cols[u].lim[ln];
    const uint32_t to = tile::lds_addr(st[s].nl) + 256 * (wave < 2 ? wave : 2);
    if constexpr (WIDE)
      tile::dma4_v(static_cast<const uint32_t*>(base) + val, to);
    else
      tile::dma4(base, val, to);
  };
  static_assert(offsetof(Stage, nd) == offsetof(Stage, nl) + 256 && offsetof(Stage, lm) == offsetof(Stage, nl) + 512, "scalars in a row");

  f32x16_t dk[NDB], dv[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      dk[db][i] = 0.f;
      dv[db][i] = 0.f;
    }
  const float sl2 = p.scale_kv_log2;

  // Fragment reads as LDS byte addresses: a per-lane base, and the d block by
  // exclusive-or (a row is a multiple of 16 * CPR bytes and the swizzle is one),
  // so that no register per block is held.
  //   rows of Q or dO: row cb*32 + l32, d = kk*16 + hf*8 ..
  //   transposed (Q^T, dO^T; d on M, columns on K) of d block db and column
  //   group j: lane (d, half) gets columns 16j + 4*half + {0..3} and + {8..11}
  //   of row d, with two transposing reads (lane r of a 16-lane group supplies
  //   row 16j + 4*half (+8) + r/4, elements d0 + 4*(r%4) .. +3); 8 rows on,
  //   bit 1 of the swizzle is the other one.
  typedef __attribute__((address_space(3))) const bf16x8_t lds_frag;
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  typedef int i32x4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) const f32x4_t lds_f4;
  typedef __attribute__((address_space(3))) const i32x4_t lds_i4;
  static_assert(sizeof(Stage) % 256 == 0, "exclusive-or on stage addresses");

  // This wavefront's 32 columns of stage S against its 32 keys; `left`:
  // columns of the step that exist.
  auto compute = [&](const Stage& S, int left, auto&& between) __attribute__((always_inline)) {
    // columns that see all of this wavefront's keys, one bit each
    const int ln = fresh_lane(), n = ln & 31, hf = ln >> 5;
    const uint64_t all = __ballot(S.lm[ln] >= key_hi && ln < left);
    const bool full = (uint32_t)(all >> (32 * cb)) == 0xffffffffu;
    const uint32_t base = tile::lds_addr(&S);
    constexpr uint32_t kG = offsetof(Stage, g);
    const int tr_r = cb * 32 + 4 * hf + ((ln & 15) >> 2), tr_c = 2 * ((ln >> 4) & 1) + ((ln & 3) >> 1);
    uint32_t b_row = base + 2 * at(cb * 32 + n, hf), b_tr = base + 2 * (at(tr_r, tr_c) + 4 * (ln & 1));
    // Before each product group: the block addresses are formed again (one
    // operation each), not kept in 16 registers from the group before.
    auto renew = [&]() __attribute__((always_inline)) { asm volatile("" : "+v"(b_row), "+v"(b_tr)); };
    const uint32_t b_col = base + (uint32_t)offsetof(Stage, nl) + 4 * (cb * 32 + hf * 4);
    // S - LSE / scale, columns on M, this wavefront's 32 keys on N: element i
    // of a lane is column (i/4)*8 + hf*4 + i%4 and key `key`.
    auto init = [&](uint32_t v) __attribute__((always_inline)) -> f32x16_t {
      f32x16_t x;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4_t f = *(lds_f4*)(uintptr_t)(v + 32 * q4);
        x[4 * q4] = f.x, x[4 * q4 + 1] = f.y, x[4 * q4 + 2] = f.z, x[4 * q4 + 3] = f.w;
      }
      return x;
    };
    auto row = [&](uint32_t blk, int kk) __attribute__((always_inline)) -> bf16x8_t {
      return *(lds_frag*)(uintptr_t)((b_row ^ (uint32_t)(kk << 5)) + blk);
    };
    auto trf = [&](uint32_t blk, int j, int db) __attribute__((always_inline)) -> bf16x8_t {
      const uint32_t to = blk + j * 32 * D;
      return tile::tr_pair_at((b_tr ^ (uint32_t)(db << 6)) + to, (b_tr ^ (uint32_t)((db << 6) | 32)) + to + 16 * D);
    };
    // The step's products in order: S (Q rows), dP (dO rows), dV (dO^T), dK
    // (Q^T), with kPre fragment reads in flight throughout, also across the
    // groups and while the first ones wait for `between` (the next loads).
    // sched_barrier keeps the compiler from requesting more at once, which
    // would not fit the registers beside the sums.
    constexpr int kPre = 3, N1 = NKK, N2 = 2 * NKK, N3 = N2 + 2 * NDB, N4 = N3 + 2 * NDB;
    auto frag = [&](auto ic) __attribute__((always_inline)) -> bf16x8_t {
      constexpr int i = decltype(ic)::value;
      if constexpr (i == N1 || i == N2 || i == N3) renew();
      if constexpr (i < N1) return row(0, i);
      else if constexpr (i < N2) return row(kG, i - N1);
      else if constexpr (i < N3) return trf(kG, (i - N2) / NDB, (i - N2) % NDB);
      else return trf(0, (i - N3) / NDB, (i - N3) % NDB);
    };
    bf16x8_t f[kPre];
    tile::static_for<kPre>([&](auto ic) __attribute__((always_inline)) { f[decltype(ic)::value] = frag(ic); });
    f32x16_t sc = init(b_col), dp;
    between();
    // P = exp(S - LSE), in place, between the dP products (the first
    // two give the last S product time to land)
    constexpr int kSlots = NKK - 1;
    bf16x8_t pb[2], sb[2], kf[2];
    tile::static_for<N4>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      if constexpr (i == N1) dp = init(b_col + 256);  // dP - D
      if constexpr (i == N2) {
        if (!full) {
          tile::static_for<4>([&](auto qc) __attribute__((always_inline)) {
            constexpr int q4 = decltype(qc)::value;
            const int r0 = cb * 32 + q4 * 8 + hf * 4;
            const i32x4_t m4 = *(lds_i4*)(uintptr_t)(b_col + 512 + 32 * q4);
            const int mv[4] = {m4.x, m4.y, m4.z, m4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) sc[4 * q4 + e] = kg * 32 + n < mv[e] && r0 + e < left ? sc[4 * q4 + e] : 0.f;
            __builtin_amdgcn_sched_barrier(0);
          });
        }
        // four elements at a time, so that P and dP give way to the operands
        tile::static_for<4>([&](auto gc) __attribute__((always_inline)) {
#pragma unroll
          for (int e = 4 * decltype(gc)::value; e < 4 * decltype(gc)::value + 4; ++e) {
            pb[e >> 3][e & 7] = (__bf16)sc[e];
            sb[e >> 3][e & 7] = (__bf16)(sc[e] * dp[e]);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
      }
      const bf16x8_t a = f[i % kPre];
      bf16x8_t kb;
      if constexpr (i >= NKR && i < N1) kb = kf[i % 2];
      // dV^T += dO^T P, dK^T += Q^T dS: d on M (block db), keys on N, columns on K
      // the LDS pieces of K, two ahead
      if constexpr (i + 2 >= NKR && i + 2 < N1) kf[i % 2] = Kl[kg][i + 2 - NKR][ln];
      if constexpr (i < NKR) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bk[i], sc, 0, 0, 0);
      else if constexpr (i < N1) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kb, sc, 0, 0, 0);
      else if constexpr (i < N2) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bv[i - N1], dp, 0, 0, 0);
      else if constexpr (i < N3) dv[(i - N2) % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[(i - N2) / NDB], dv[(i - N2) % NDB], 0, 0, 0);
      else dk[(i - N3) % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, sb[(i - N3) / NDB], dk[(i - N3) % NDB], 0, 0, 0);
      if constexpr (i + kPre < N4) f[i % kPre] = frag(std::integral_constant<int, i + kPre>{});
      if constexpr (i > N1 && i < N2) {
        constexpr int p0 = i - N1 - 1;
#pragma unroll
        for (int e = 16 * p0 / kSlots; e < 16 * (p0 + 1) / kSlots; ++e) sc[e] = fast_exp2(sc[e] * sl2);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Step t computes stage t % 3, loaded at step t-2, and loads the columns of
  // step t+2 into the stage of step t-1, which every wavefront has read
  // before this step's barrier; their list was written at step t-1.  Wavefront
  // 7 writes the list of step t+3 now, from the query rows it fetched at step
  // t-1, and fetches those of step t+4 to where list t was, which was read at
  // step t-2.  Before the barrier each wavefront waits for its own loads of
  // step t and wavefront 7 for its list's stores; at most the 2*IPW+1 loads of
  // step t+1 are still in flight (the rows were fetched before them).
  const int n_steps = (c_end - c_begin + COLS - 1) / COLS;
  if (wave == 7) {
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      fetch_rows(u);
      tile::wait_vm<0>();
      asm volatile("" ::: "memory");
      list_rows(u);
    }
    fetch_rows(3);
  }
  // K and V are waited for here: pending into the loop, their waits there
  // would be for every load in flight.
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    asm volatile("" : "+v"(bv[kk]));
    if (kk < NKR) asm volatile("" : "+v"(bk[kk]));
  }
  __syncthreads();
  load(0, 0);
  load(1, 1);
  int s = 0, left = c_end - c_begin;
  for (int t = 0; t < n_steps; ++t, left -= COLS) {
    tile::wait_vm<2 * IPW + 1>();
    if (wave == 7) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    tile::bar();
    auto feed = [&]() __attribute__((always_inline)) {
      if (wave == 7) {
        list_rows((t + 3) & 3);
        fetch_rows(t & 3);
      }
      load((t + 2) & 3, s == 0 ? 2 : s - 1);
    };
    if (idle)
      feed();
    else
      compute(st[s], left, feed);
    s = s == 2 ? 0 : s + 1;
  }
  __builtin_amdgcn_s_waitcnt(0);
  tile::bar();  // no load in flight, no stage in use

  // The two column halves of a key group add up through LDS: wavefronts 0-3
  // end with dK of their keys, wavefronts 4-7 with dV, 64 dims at a time.
  f32x16_t* xch = reinterpret_cast<f32x16_t*>(smem);  // [tensor][kg][db % 2][lane]
#pragma unroll
  for (int h = 0; h < NDB / 2 + NDB % 2; ++h) {
    if (h) __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x)
      if (2 * h + x < NDB) xch[((cb * 4 + kg) * 2 + x) * 64 + lane] = cb ? dk[2 * h + x] : dv[2 * h + x];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x)
      if (2 * h + x < NDB) {
        const f32x16_t o = xch[(((cb ^ 1) * 4 + kg) * 2 + x) * 64 + lane];
        if (cb)
          dv[2 * h + x] += o;
        else
          dk[2 * h + x] += o;
      }
  }
  if (key >= b.n_keys) return;
  // element i of block db: d = db*32 + (i/4)*8 + hf*4 + i%4, key `key`.  An item
  // that holds all of its key run's columns writes its rows, a piece of a
  // split run its slot's (the sums follow in bwd_reduce_kernel).
  const float scl = cb ? 1.f : p.scale;
  const int32_t slot = b.cost;
  if (slot < 0) {
    uint16_t* dst = static_cast<uint16_t*>(cb ? p.dv : p.dk) + ((b.key_row0 + key) * Hkv + kvh) * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = (cb ? dv[db][4 * i4 + e] : dk[db][4 * i4 + e]) * scl;
        uint2 pk;
        pk.x = (uint32_t)f32_to_bf16_bits(x[0]) | ((uint32_t)f32_to_bf16_bits(x[1]) << 16);
        pk.y = (uint32_t)f32_to_bf16_bits(x[2]) | ((uint32_t)f32_to_bf16_bits(x[3]) << 16);
        *reinterpret_cast<uint2*>(dst + db * 32 + i4 * 8 + hf * 4) = pk;
      }
  } else {
    float* dst = p.part + (((int64_t)slot * 2 + cb) * kBwdKeys + key) * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = (cb ? dv[db][4 * i4 + e] : dk[db][4 * i4 + e]) * scl;
        *reinterpret_cast<float4*>(dst + db * 32 + i4 * 8 + hf * 4) = make_float4(x[0], x[1], x[2], x[3]);
      }
  }
}

// ------------------------------------------------------------------ sums

// dK and dV rows of split key runs: the pieces' sums added in their order
// (so results do not depend on scheduling) and rounded to bf16 (nearest
// even); and zero rows where no query sees a key.  One workgroup per 16 rows
// of a record: a copy, 16 bytes a lane, a piece's loads in flight together.
template <int D>
__global__ __launch_bounds__(256) void bwd_reduce_kernel(BwdParams p) {
  constexpr int kRows = 16, kParts = kBwdKeys / kRows, Q = D / 4;
  const BwdReduce r = load_scalar(p.breduce + blockIdx.x / kParts);
  const int k0 = (blockIdx.x % kParts) * kRows;
  if (k0 >= r.n_keys) return;
  const int rows = min(kRows, r.n_keys - k0);
  if (r.n_slots == 0) {
    // rows k0 .. of all heads, contiguous
    uint2* dk = reinterpret_cast<uint2*>(p.dk) + (r.row0 + k0) * p.Hkv * Q;
    uint2* dv = reinterpret_cast<uint2*>(p.dv) + (r.row0 + k0) * p.Hkv * Q;
    for (int64_t i = threadIdx.x; i < (int64_t)rows * p.Hkv * Q; i += 256) dk[i] = dv[i] = make_uint2(0, 0);
    return;
  }
  for (int i = threadIdx.x; i < 2 * rows * Q; i += 256) {
    const int t = i / (rows * Q), e = i % (rows * Q), key = k0 + e / Q, c = e % Q;
    const float4* src = reinterpret_cast<const float4*>(p.part) + (((int64_t)r.slot0 * 2 + t) * kBwdKeys + key) * Q + c;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int s = 0; s < r.n_slots; ++s) {
      const float4 x = src[(int64_t)s * 2 * kBwdKeys * Q];
      a.x += x.x, a.y += x.y, a.z += x.z, a.w += x.w;
    }
    uint2 pk;
    pk.x = (uint32_t)f32_to_bf16_bits(a.x) | ((uint32_t)f32_to_bf16_bits(a.y) << 16);
    pk.y = (uint32_t)f32_to_bf16_bits(a.z) | ((uint32_t)f32_to_bf16_bits(a.w) << 16);
    uint16_t* dst = static_cast<uint16_t*>(t ? p.dv : p.dk) + ((r.row0 + key) * p.Hkv + r.kvh) * D;
    reinterpret_cast<uint2*>(dst)[c] = pk;
  }
}

template <int D>
void launch_dkdv(const BwdParams& p, int n_bwd, hipStream_t stream) {
  if (std::max(p.n_q * p.Hq * D * 2, p.n_btok * 4) < (int64_t)1 << 32)
    hipLaunchKernelGGL((bwd_dkdv_kernel<D, false>), dim3(n_bwd), dim3(kThreads), 0, stream, p);
  else
    hipLaunchKernelGGL((bwd_dkdv_kernel<D, true>), dim3(n_bwd), dim3(kThreads), 0, stream, p);
}

}  // namespace

hipError_t launch_tree_attn_bwd(const BwdParams& p, int n_work, int n_bwd, int D, hipStream_t stream) {
  const dim3 blk256(256);
  if (p.n_btokens > 0)
    hipLaunchKernelGGL(bwd_tokens_kernel, dim3((unsigned)((p.n_btokens + 3) / 4)), blk256, 0, stream, p);
  if (n_work > 0) {
    if (D == 64)
      hipLaunchKernelGGL((bwd_dq_kernel<64>), dim3(n_work), dim3(kThreads), 0, stream, p);
    else
      hipLaunchKernelGGL((bwd_dq_kernel<128>), dim3(n_work), dim3(kThreads), 0, stream, p);
  }
  if (n_bwd > 0) {
    if (D == 64)
      launch_dkdv<64>(p, n_bwd, stream);
    else
      launch_dkdv<128>(p, n_bwd, stream);
  }
  if (p.n_breduce > 0) {
    const dim3 grid((unsigned)p.n_breduce * (kBwdKeys / 16));
    if (D == 64)
      hipLaunchKernelGGL((bwd_reduce_kernel<64>), grid, blk256, 0, stream, p);
    else
      hipLaunchKernelGGL((bwd_reduce_kernel<128>), grid, blk256, 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace padoc
