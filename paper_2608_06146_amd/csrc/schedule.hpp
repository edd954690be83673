// Device-side schedule records and kernel parameter blocks.
//
// The planner (host/plan.cpp) serialises these records into the caller's
// workspace; the kernels read them.  The record layouts are the ones the C
// ABI exports for inspection (padoc_work_view / padoc_range_view).
#pragma once

#include <stdint.h>

#include "padoc_attn.h"  // include/ is on the include path

namespace padoc {

using WorkRec = padoc_work_view;    // 48 bytes
using RangeRec = padoc_range_view;  // 32 bytes
using BwdRec = padoc_bwd_view;      // 40 bytes
static_assert(sizeof(WorkRec) == 48, "work record is 48 bytes");
static_assert(sizeof(RangeRec) == 32, "range record is 32 bytes");
static_assert(sizeof(BwdRec) == 40, "backward record is 40 bytes");

// Key tile of every kernel (keys staged per step) and columns per work item.
constexpr int kTileKeys = 64;
constexpr int kTileCols = 256;
constexpr int kBlock = 16;  // paged KV block (tokens)
constexpr int kPrivateCols = 16;  // columns of a private decode item (one wavefront)
constexpr int kPrivateQueues = 8;  // decode: private item queues (one per XCD)
constexpr int kBwdKeys = 128;     // keys of a backward key-major item (4 x 32)
constexpr int kMaxItemKeys = 8192;  // decode: keys of a chunk (item) at most
constexpr int kMaxItemTiles = kMaxItemKeys / kTileKeys;  // tiles of a paged tile item at most

// Backward schedule records that only the device reads.  A BwdRec on the
// device holds in `cost` the partial slot its item writes (-1: the item has
// all columns of its key run and writes the run's dK / dV rows).
struct BwdTokens {  // tokens dst .. dst+count-1 of the items' token lists:
  int32_t dst, row0, count;  // query row row0 + i,
  int32_t lim0, slope, lim_max;  // limit min(lim0 + slope * i, lim_max)
};
struct BwdReduce {  // n_slots > 0: rows = sum of the slots; 0: n_keys rows of every head are zero
  int64_t row0;
  int32_t n_keys, kvh, slot0, n_slots;
};
static_assert(sizeof(BwdTokens) == 24 && sizeof(BwdReduce) == 24, "device records");

// Everything a tile kernel needs.  Pointers are device pointers.
struct TileParams {
  const void* q;          // [n_q, Hq, D]
  const void* k;          // packed [T, Hkv, D] or paged [blocks, Hkv, 16, D]
  const void* v;
  void* o;                // final mode: [n_q, Hq, D]
  float* lse;             // final mode: [n_q, Hq]
  const int32_t* block_table;  // paged mode
  const WorkRec* work;
  const RangeRec* ranges;
  const RangeRec* first;      // decode, bf16: first range of tile item i, its tiles counted in `reserved`
  const int32_t* lims;
  const int32_t* toks;
  float* part_o;          // partial mode: [slots, D] unnormalised accumulators
  float* part_ml;         // partial mode: [slots, 2] (running max in log2 units, sum)
  int32_t Hq, Hkv, G;
  float scale_log2;       // softmax_scale * log2(e)
};

// Backward of the packed forward (bf16).
struct BwdParams {
  const void* q;     // [n_q, Hq, D]
  const void* k;     // [T, Hkv, D]
  const void* v;
  const void* o;     // [n_q, Hq, D]
  const float* lse;  // [n_q, Hq]
  const void* dout;  // [n_q, Hq, D]
  void* dq;          // [n_q, Hq, D]
  void* dk;          // [T, Hkv, D]
  void* dv;
  float* nd;         // workspace [n_q, Hq]: -sum_d dout * o
  float* nl;         // workspace [n_q, Hq]: -lse / scale_kv
  float* part;       // workspace [slots][2: dK, dV][kBwdKeys][D] fp32: sums of the pieces of split key runs
  const WorkRec* work;  // the forward's query-major items (dQ)
  const RangeRec* ranges;
  const int32_t* lims;
  const int32_t* toks;
  const BwdRec* bwd;    // key-major items (dK, dV)
  int32_t* btoks;       // workspace, written from btokens
  int32_t* blims;
  const BwdTokens* btokens;
  const BwdReduce* breduce;
  int64_t n_q, T, n_btok;
  int32_t n_btokens, n_breduce;
  int32_t Hq, Hkv, G;
  float scale, scale_log2;
  // dK/dV: its scores start at -lse / scale, so its scale is at least 1e-36,
  // where that stays finite (at smaller ones, scale * q.k up to q.k = 1e28 is
  // below fp32's last bit beside lse).
  float scale_kv, scale_kv_log2;
};

struct CombineParams {
  const int32_t* comb_slot;  // partial slots, grouped by (row, KV head)
  const int4* comb_rows;     // per merged pair: {row*Hkv + kvh, first, end, 0} into comb_slot
  int64_t n_rows;
  const float* part_o;
  const float* part_ml;
  void* o;
  float* lse;
  int64_t n_q;
  int32_t Hq, Hkv, G;
  int32_t* next;  // decode: the step kernel's kPrivateQueues queue counters (256 bytes apart), zeroed for the next call
};

}  // namespace padoc
