// Launch interfaces between the C-ABI layer and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "attn_schedule.h"
#include "step_rules.h"

namespace racer {

// Device counters (unsigned long long each)
enum Counter : int {
  kCtrLookups = 0, kCtrHits, kCtrMisses, kCtrUnique, kCtrInserted, kCtrEvicted, kCtrBypassed,
  kCtrInvalid, kCtrShrinkEvicted, kCtrShrinkMoved, kCtrBadPages, kCtrUnorderedTs, kCtrCount
};

// The counters exist in kCtrShards copies; a block adds to the copy chosen by its index so that
// thousands of blocks do not serialise on one address.  pool_stats adds the copies up.
constexpr int kCtrShards = 64;
#if defined(__HIPCC__)
__device__ __forceinline__ int ctr_index(int counter) { return static_cast<int>(blockIdx.x & (kCtrShards - 1)) * kCtrCount + counter; }
#endif

// One embedding table behind the pool.  With several tables a row is known by its global id, base + row; rows
// narrower than the pool's slots are kept zero-padded.
struct TableDesc {
  uint64_t base, rows;
  const uint8_t* ptr;  // device-visible address of the pinned host rows
  uint32_t row_bytes, pad;
};
constexpr uint32_t kMaxTables = 32;

// Everything a kernel needs to find a cache set, its ways and its rows.
// Way layer w of the cache = slot w of every set = `layer_pages` consecutive logical EMB
// pages; slot (w, s) lives in logical page w*layer_pages + s/spp at offset s%spp.
struct EmbView {
  uint8_t* base;            // pool backing store
  uint64_t page_size;
  uint32_t row_bytes;
  uint32_t spp;             // slots per page
  uint32_t w_max;
  uint32_t elem;            // 0 fp32, 1 bf16
  uint32_t sets;
  uint32_t layer_pages;
  uint32_t full_ways;       // n_emb / layer_pages
  uint32_t part_sets;       // (n_emb % layer_pages) * spp: these sets have one more way
  uint32_t* tags;           // [sets][w_max]
  uint32_t* stamps;         // [sets][w_max]
  const int32_t* emb_pages; // logical -> physical page
  const uint8_t* table;     // device-visible address of the pinned host table
  uint64_t rows;            // rows of all tables together
  const TableDesc* tables;  // more than one table: their descriptors, bases ascending (else nullptr)
  uint32_t n_tables;
  unsigned long long* counters;
};

// Lookup ids: int64 row numbers, or (table, row) pairs when table_of is set.
struct IdSrc {
  const int64_t* ids;
  const uint32_t* table_of;
};

// Entry of the dedupe table: key = (batch << 32) | id, val = (batch << 32) | (0xFFFFFFFF - first lookup index).
struct HashEnt {
  unsigned long long key, val;
};

// Scratch of the miss path.  A probe block lists what it finds in its own stretch of the lists: block b owns
// [b * seg, (b + 1) * seg) of the per-lookup arrays.  Tables are keyed by the batch number, so nothing is cleared
// between calls on one pool.
constexpr uint32_t kMinStretch = 32;  // lookups per probe block at the least
struct MissWs {
  uint32_t seg;             // lookups per probe block (set by the probe's launch)
  uint32_t* any;            // = batch when some block of the batch had a miss
  uint32_t* seg_cnt;        // per stretch: (waiting output rows << 16) | new ids
  uint32_t* def_list;       // output rows that wait for a miss
  int64_t* loc;             // per lookup of a waiting row: >=0 pool byte offset, -1 zero row, <=-3 dedupe slot -(v+3)
  HashEnt* hents;
  uint32_t* hslot_u;        // number of the new id in a dedupe slot
  uint32_t hmask;
  unsigned long long* heads;  // per-set chains of new ids: (batch << 32) | number
  uint32_t headmask;
  uint4* rec;               // per new id: id, set, next in the chain (0xFFFFFFFF: last), dedupe slot
  int32_t* u_way;           // the way it takes, -1: none
  uint8_t* staging;         // its row, fetched from the host table
};

// probe, hit gather, missing rows fetched into staging; sets ws.seg for the miss path that follows
hipError_t launch_emb_probe(const EmbView& v, MissWs& ws, const IdSrc& ids, uint32_t n, uint32_t bag, uint8_t* out,
                            uint8_t* hit_flags, uint32_t batch, hipStream_t stream);
// cache insertion of the new ids and the output rows that waited for them
hipError_t launch_emb_miss_path(const EmbView& v, const MissWs& ws, uint32_t n, uint32_t bag, uint8_t* out, uint32_t batch,
                                hipStream_t stream);

// refill of empty ways with `ids` (hottest first): probe, then the miss path restricted to empty ways
hipError_t launch_emb_refill(const EmbView& v, MissWs ws, const IdSrc& ids, uint32_t n, uint32_t batch, hipStream_t stream);

hipError_t launch_emb_shrink(const EmbView& v, uint32_t old_full, uint32_t old_part_sets,
                             hipStream_t stream);

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t value, hipStream_t stream);

// measurement aid: n_reads reads of random rows (128, 256, 512 or 1024 bytes) out of n_rows rows at `base`,
// written out back to back at `out` unless that is null
hipError_t launch_random_row_reads(const void* base, uint64_t n_rows, uint32_t row_bytes, uint64_t n_reads, void* out,
                                   uint64_t seed, hipStream_t stream);

// ---- HSTU -----------------------------------------------------------------------------
struct HstuDims {
  uint32_t L, d, H, dh, elem, pt, n_pos, n_time;
  float inv_n, eps;
  uint32_t pt_shift;  // log2(pt) when pt is a power of two, else 32
};

struct KvView {
  uint8_t* base;
  uint64_t page_size;
  uint32_t n_pages;
  unsigned long long* counters;
};

// What a workgroup of the fp32 attention does: 16 queries of one request
constexpr uint32_t kF32Queries = 16;
struct F32Tile {
  uint32_t req, q0;
};

// Up to 128 consecutive new-token rows of one request (projection GEMM tile)
struct RowTile {
  uint32_t row0, rows, req, pad;
};

// Where each die's attention work lies in the work list: block i does entry begin[i % kXcds] + i / kXcds
struct AttnDies {
  uint32_t begin[kXcds + 1];
  uint32_t piece;  // key tiles of a piece (of query tiles that are cut)
};

// Work lists built on the host for one step
struct StepLists {
  const ReqDev* reqs;          // [B]
  const uint32_t* ts_marks;    // [B] = epoch where the request's timestamps decrease somewhere
  uint32_t epoch;
  // bf16 models (attn_schedule.h)
  const AttnItem* items;
  const AttnWork* work;
  AttnDies dies;
  uint32_t n_blocks;
  bool turns;                  // the blocks of a CU take turns at going first
  const uint32_t* groups;      // query tiles whose partial outputs are to be added up
  uint32_t n_groups;
  bool sum_rows;               // by attention_reduce_rows (step_rules.h)
  float* partials;             // [slot][128][64]
  const RowTile* row_tiles;    // projection tiles, none crosses a request
  uint32_t n_row_tiles;
  const uint32_t* group_req;   // request of rows 0, 32, .. and, behind the last of these, of the last row
  const F32Tile* f32_tiles;    // fp32 models
  uint32_t n_f32_tiles;
  uint32_t longest;            // tokens of the longest request, cached ones included
  uint64_t f32_keys;           // keys that the fp32 tiles see, all together
  uint32_t B, N;
};

// Lists of up to this size are handed to the kernel that begins a step as an argument.
constexpr uint32_t kListArgBytes = 3072;
struct ListArg {
  alignas(16) uint8_t bytes[kListArgBytes];
};

// Begins a step: one pass over every request's timestamps (max_seq: the longest request's prefix + new tokens); a request
// whose timestamps decrease somewhere is marked with the step's epoch and counted in kCtrUnorderedTs.  The
// attention kernels take their 32-bit relative-time paths only for ordered requests (an unordered one gets the general
// 64-bit gaps, where a negative gap falls into bucket 0).  The kernel also writes the lists (list_bytes, a multiple of 16)
// to list_dst: out of its argument if there is one, else from pinned host memory.
hipError_t launch_begin_step(const StepLists& sl, uint32_t max_seq, const int64_t* ts, unsigned long long* counters, const ListArg* arg,
                             const uint8_t* pinned, uint8_t* list_dst, uint64_t list_bytes, hipStream_t stream);

hipError_t launch_layernorm(const HstuDims& hd, const void* x, const float* g, const float* b,
                            const void* gate /*nullable: multiply by gate rows*/, void* y, uint32_t N,
                            hipStream_t stream);
hipError_t launch_gemm_front(const HstuDims& hd, uint32_t layer, const void* xn, const void* w1t,
                             const float* b1, void* u, void* q, const KvView& kv, const StepLists& sl,
                             const int32_t* page_tables, hipStream_t stream);
hipError_t launch_gemm_back(const HstuDims& hd, const void* g, const void* w2t, const float* b2,
                            const void* x, void* y, uint32_t N, hipStream_t stream);
// bf16 models with d = 64, 128, 256 or 512: LayerNorm, projection and epilogue of a layer half in one kernel
// (front: X -> U, Q*log2(e), K/V pages; back: O, U, X -> Y); weights as fragments.
// In bf16 models U, O, the normalised matrices and the library's weight copies (launch_weight_copy) are half precision.
bool layer_halves_fused(const HstuDims& hd);
hipError_t launch_layer_front_fused(const HstuDims& hd, uint32_t layer, const void* x, const float* ln_g,
                                    const float* ln_b, const void* w1f, const float* b1, void* u, void* q,
                                    const KvView& kv, const StepLists& sl, const int32_t* page_tables,
                                    hipStream_t stream);
hipError_t launch_layer_back_fused(const HstuDims& hd, const void* o, const void* u, const float* ln_g,
                                   const float* ln_b, const void* w2f, const float* b2, const void* x, void* y,
                                   const StepLists& sl, hipStream_t stream);
// Small steps of such models: a back half and the next layer's front half in one kernel, or one of them alone (the other
// null).  x: the back half's residual, or what a front half alone takes.  The front's u must not be the back's.
struct LayerBack { const void *o, *u; const float *ln_g, *ln_b; const void* w2f; const float* b2; void* y; };
struct LayerFront { uint32_t layer; const float *ln_g, *ln_b; const void* w1f; const float* b1; void *u, *q; };
bool layers_joined(const HstuDims& hd, uint32_t N, uint32_t B, uint64_t cached);  // N new tokens of B requests behind `cached` ones
// begin: the first front half's kernel also begins the step (as launch_begin_step with an argument), which it does where
// begin_joins says so: with up to 512 blocks' worth of timestamps, which find room beside the rows'.
struct BeginStep {
  const ListArg* arg;
  uint32_t max_seq;
  const int64_t* ts;
  unsigned long long* counters;
  uint8_t* list_dst;
  uint64_t list_bytes;
};
bool begin_joins(const StepLists& sl, uint32_t max_seq);
hipError_t launch_layer_join(const HstuDims& hd, const LayerBack* back, const LayerFront* front, const void* x, const KvView& kv,
                             const StepLists& sl, const int32_t* page_tables, hipStream_t stream, const BeginStep* begin = nullptr);
// o_half (bf16 models): the output is written in half precision (the step's own matrix between the attention and the
// second LayerNorm) instead of bf16 (what a caller of the attention alone gets)
hipError_t launch_attention(const HstuDims& hd, uint32_t layer, const void* q, const float* pos,
                            const float* time, const KvView& kv, const StepLists& sl,
                            const int32_t* page_tables, const int64_t* ts, void* o, bool o_half, hipStream_t stream);
// adds up the fp32 partials of query tiles cut into pieces (no-op when none was)
hipError_t launch_attention_reduce(const HstuDims& hd, const StepLists& sl, void* o, bool o_half, hipStream_t stream);
// bf16 models: pos and time must be the tables multiplied by log2(e) (launch_scale_bias), and
// q must already be multiplied by log2(e) (the front halves store it that way)
hipError_t launch_scale_bias(const float* in, float* out, uint64_t n, hipStream_t stream);
hipError_t launch_scale_q(const void* in, void* out, uint64_t n, hipStream_t stream);
// the library's half-precision copy of a bf16 weight matrix: transposed, or (fragments) in the operand order of the fused
// layer halves
hipError_t launch_weight_copy(const void* w, void* wt, uint32_t rows, uint32_t cols, bool fragments, hipStream_t stream);

// fp32 models: a layer half in one kernel (front: in = X -> U, Q, K/V pages; back: in = O, gate = U, resid = X -> Y), W as
// the caller gave it, and the attention
hipError_t launch_layer_half_f32(const HstuDims& hd, uint32_t layer, bool front, const float* in, const float* gate, const float* ln_g,
                                 const float* ln_b, const float* w, const float* bias, float* u, float* q, const KvView& kv,
                                 const StepLists& sl, const int32_t* page_tables, const float* resid, float* y, hipStream_t stream);
hipError_t launch_attention_f32(const HstuDims& hd, uint32_t layer, const float* q, const float* pos, const float* time, const KvView& kv,
                                const StepLists& sl, const int32_t* page_tables, const int64_t* ts, float* o, hipStream_t stream);

}  // namespace racer
