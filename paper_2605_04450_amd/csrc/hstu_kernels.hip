// HSTU layer kernels of bf16 models for gfx950 (paper Sec. II-A/II-B "Compute" stage; the layer equations
// are the published HSTU form):
//   Xn = LayerNorm(X);  [U|V|Q|K] = SiLU(Xn W1 + b1);  K,V of the new tokens -> KV pages
//   O_i = (1/n) sum_{j<=p_i} SiLU(q_i.k_j + pos[min(p_i-j, n_pos-1)] + time[bucket(ts_p-ts_j)]) v_j
//   Y = X + (LayerNorm(O) * U) W2 + b2
// They run on MFMA with fp32 accumulation (fp32 models: hstu_fp32.hip).
// What a bf16 model stores where a caller can see it (inputs, weights, K and V in the pages, outputs) is bf16.
// The library's own intermediate matrices (the normalised activations, U, the attention output O, the gated
// activations) and its copies of the weights (MFMA operand fragments for the fused layer halves, transposed for the other
// widths) are IEEE half precision: eleven significant bits instead of eight at the same size and the same MFMA rate
// (v_mfma_f32_32x32x16_f16), which halves the
// distance to the fp64 oracle; a bf16 weight converts exactly.  Values of these matrices must stay below
// 65504 in magnitude, which LayerNorm and the 1/n scaling ensure for any sane model.  The two attention
// products take bf16 operands (Q, and K, V as the pages hold them).
//
// KV page layout (one page = page_tokens tokens of every layer):
//   [layer][K|V][head] blocks of page_tokens*d_h elements;
//   a K block is [token][d_h]; a V block is stored transposed, [d_h][token], so that the
//   second product's matrix operand (contraction over keys) is read key-contiguous.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "hstu_common.h"

namespace racer {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct bf16_t { uint16_t bits; };
struct half_t { uint16_t bits; };  // IEEE binary16 (the library's own intermediates)
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // like uint4, but a value that stays in registers
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return static_cast<uint16_t>((u >> 16) | 0x40);
  return static_cast<uint16_t>((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ uint16_t f2h(float f) { return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f)); }  // nearest even
// ---------------------------------------------------------------------------------------
// LayerNorm over d (optionally times a gate row), two-pass in fp32.  A row is owned by LPR
// consecutive lanes of a wavefront (64 / LPR rows per wavefront, LPR chosen so that every
// lane has work); a lane holds KC chunks of 8 consecutive elements (16-byte accesses for
// bf16), d <= 1024.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void load8(const float* p, float v[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t* p, float v[8]) {
  const uint4 a = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[2 * k] = __uint_as_float(w[k] << 16);
    v[2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ void load8(const half_t* p, float v[8]) {
  const uint4 a = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const f16x2 h = __builtin_bit_cast(f16x2, w[k]);
    v[2 * k] = static_cast<float>(h[0]);
    v[2 * k + 1] = static_cast<float>(h[1]);
  }
}
__device__ __forceinline__ uint32_t pack2_f16(float lo, float hi) {
  typedef float v2f __attribute__((ext_vector_type(2)));
  const v2f v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}
__device__ __forceinline__ void store8(half_t* p, const float v[8]) {
  *reinterpret_cast<uint4*>(p) = make_uint4(pack2_f16(v[0], v[1]), pack2_f16(v[2], v[3]), pack2_f16(v[4], v[5]), pack2_f16(v[6], v[7]));
}
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {  // sum over the LPR lanes that share a row
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <typename TX, typename TY, int LPR, int KC>  // TX: input rows; TY: gate rows and output rows
__global__ __launch_bounds__(256) void layernorm_rows(const TX* __restrict__ x, const float* __restrict__ g,
                                                      const float* __restrict__ b, const TY* __restrict__ gate,
                                                      TY* __restrict__ y, uint32_t N, uint32_t d, float eps) {
  const uint32_t sub = threadIdx.x % LPR;
  const uint32_t row = blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
  const bool row_ok = row < N;  // lanes of a missing row still take part in the shuffles
  const uint32_t chunks = d / 8;
  const uint64_t base = static_cast<uint64_t>(row_ok ? row : 0) * d;
  float v[KC][8], gt[KC][8];
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    const uint32_t c = sub + LPR * k;
    const bool on = row_ok && c < chunks;
    if (on) load8(x + base + 8 * c, v[k]);
    if (on && gate) load8(gate + base + 8 * c, gt[k]);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (!on) v[k][e] = 0.0f;
  }
  float s = 0.0f;
#pragma unroll
  for (int k = 0; k < KC; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) s += v[k][e];
  const float mean = group_sum<LPR>(s) / d;
  float q = 0.0f;
#pragma unroll
  for (int k = 0; k < KC; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float dv = (sub + LPR * k < chunks) ? v[k][e] - mean : 0.0f;
      q += dv * dv;
    }
  const float rstd = 1.0f / sqrtf(group_sum<LPR>(q) / d + eps);
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    const uint32_t c = sub + LPR * k;
    if (!row_ok || c >= chunks) continue;
    float gg[8], bb[8], o[8];
    load8(g + 8 * c, gg);
    load8(b + 8 * c, bb);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (v[k][e] - mean) * rstd * gg[e] + bb[e];
    if (gate) {
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] *= gt[k][e];
    }
    store8(y + base + 8 * c, o);
  }
}

// ---------------------------------------------------------------------------------------
// Half-precision GEMM on MFMA (both operands are the library's own: a normalised activation matrix and a
// transposed weight copy): Y = X + A Bt^T + b2 with A [M][K] and Bt [K][K], block tile 128 x 64, four
// wavefronts of 32 rows x 64 columns each, K staged through LDS 64 at a time.
// Operand layout of v_mfma_f32_32x32x16_f16 / _bf16: lane (g = lane/32, i = lane%32) supplies row
// (A) or column (B) i with eight consecutive k of its half g; the result lane holds column
// i and rows 8*(r/4) + 4*g + r%4 for r = 0..15.
// ---------------------------------------------------------------------------------------
constexpr int kLdsPad = 8;

__global__ __launch_bounds__(256) void gemm_back_bf16(const uint16_t* __restrict__ A, const uint16_t* __restrict__ Bt, uint32_t M,
                                                      uint32_t K, const float* __restrict__ b2, const uint16_t* __restrict__ x,
                                                      uint16_t* __restrict__ y) {
  __shared__ __attribute__((aligned(16))) uint16_t As[128][64 + kLdsPad];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[64][64 + kLdsPad];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5, li = lane & 31;
  const uint32_t m0 = blockIdx.x * 128, n0 = blockIdx.y * 64;
  f32x16 acc[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;

  for (uint32_t k0 = 0; k0 < K; k0 += 64) {
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const uint32_t c = tid + 256 * it, row = c >> 3, part = c & 7;
      uint4 val = make_uint4(0, 0, 0, 0);
      if (m0 + row < M) val = *reinterpret_cast<const uint4*>(A + static_cast<uint64_t>(m0 + row) * K + k0 + part * 8);
      *reinterpret_cast<uint4*>(&As[row][part * 8]) = val;
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const uint32_t c = tid + 256 * it, row = c >> 3, part = c & 7;
      *reinterpret_cast<uint4*>(&Bs[row][part * 8]) =
          *reinterpret_cast<const uint4*>(Bt + static_cast<uint64_t>(n0 + row) * K + k0 + part * 8);
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const f16x8 a = __builtin_bit_cast(f16x8, *reinterpret_cast<const uint4*>(&As[32 * wave + li][16 * st + 8 * g]));
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        const f16x8 b = __builtin_bit_cast(f16x8, *reinterpret_cast<const uint4*>(&Bs[32 * cb + li][16 * st + 8 * g]));
        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc[cb], 0, 0, 0);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t row = m0 + 32 * wave + 8 * (r / 4) + 4 * g + (r % 4);
      if (row >= M) continue;
      const uint32_t col = n0 + 32 * cb + li;
      const uint64_t i = static_cast<uint64_t>(row) * K + col;  // (square: as many columns out as in)
      y[i] = f2bf(bf2f(x[i]) + acc[cb][r] + b2[col]);
    }
}

// ---------------------------------------------------------------------------------------
// Pointwise projection of bf16 models: [U|V|Q|K] = SiLU(Xn W1 + b1) on MFMA, one block per
// (row tile, 64 output columns).  Row tiles never cross a request (host-built list), and 64
// columns are exactly one head's slice of U, V, Q or K, so a block has one destination:
// the results go through LDS and leave as 16-byte stores - rows of U/Q, token rows of the K
// block, and key-contiguous runs of the transposed V block.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gemm_front_bf16(HstuDims hd, uint32_t layer, const uint16_t* __restrict__ A,
                                                       const uint16_t* __restrict__ Bt, const float* __restrict__ b1,
                                                       uint16_t* __restrict__ u, uint16_t* __restrict__ q, KvView kv,
                                                       const ReqDev* __restrict__ reqs,
                                                       const RowTile* __restrict__ row_tiles,
                                                       const int32_t* __restrict__ page_tables) {
  __shared__ __attribute__((aligned(16))) uint16_t As[128][64 + kLdsPad];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[64][64 + kLdsPad];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 5, li = lane & 31;
  const RowTile rt = row_tiles[blockIdx.x];
  const uint32_t m0 = rt.row0, rows = rt.rows, n0 = blockIdx.y * 64, K = hd.d;
  f32x16 acc[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;
  for (uint32_t k0 = 0; k0 < K; k0 += 64) {
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const uint32_t c = tid + 256 * it, row = c >> 3, part = c & 7;
      uint4 val = make_uint4(0, 0, 0, 0);
      if (row < rows) val = *reinterpret_cast<const uint4*>(A + static_cast<uint64_t>(m0 + row) * K + k0 + part * 8);
      *reinterpret_cast<uint4*>(&As[row][part * 8]) = val;
    }
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const uint32_t c = tid + 256 * it, row = c >> 3, part = c & 7;
      *reinterpret_cast<uint4*>(&Bs[row][part * 8]) =
          *reinterpret_cast<const uint4*>(Bt + static_cast<uint64_t>(n0 + row) * K + k0 + part * 8);
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const f16x8 a = __builtin_bit_cast(f16x8, *reinterpret_cast<const uint4*>(&As[32 * wave + li][16 * st + 8 * g]));
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        const f16x8 b = __builtin_bit_cast(f16x8, *reinterpret_cast<const uint4*>(&Bs[32 * cb + li][16 * st + 8 * g]));
        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc[cb], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  // ---- epilogue: bias + SiLU (+ log2 e for Q) -> bf16 tile in LDS (reusing As) ----
  const uint32_t which = n0 / hd.d, head = (n0 % hd.d) / 64;  // 0 U, 1 V, 2 Q, 3 K
  const float qscale = which == 2 ? 1.4426950408889634f : 1.0f;
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    const float bias = b1[n0 + 32 * cb + li];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const uint32_t row = 32 * wave + 8 * (r / 4) + 4 * g + (r % 4);
      const float z = silu(acc[cb][r] + bias) * qscale;
      As[row][32 * cb + li] = which == 0 ? f2h(z) : f2bf(z);  // U is the library's own (half precision); Q, K, V are bf16
    }
  }
  __syncthreads();
  if (which == 0 || which == 2) {
    uint16_t* dst = which == 0 ? u : q;
    for (uint32_t idx = tid; idx < 128 * 8; idx += 256) {
      const uint32_t row = idx >> 3, part = idx & 7;
      if (row < rows)
        *reinterpret_cast<uint4*>(dst + static_cast<uint64_t>(m0 + row) * hd.d + head * 64 + part * 8) =
            *reinterpret_cast<const uint4*>(&As[row][part * 8]);
    }
    return;
  }
  const ReqDev rq = reqs[rt.req];
  const uint32_t pos0 = rq.prefix_len + (m0 - rq.x_off);  // sequence position of the tile's first row
  if (which == 3) {  // K block: [token][d_h], one 128-byte row per token
    const uint64_t koff = kv_block_offset(hd, layer, 0, head, 2);
    for (uint32_t idx = tid; idx < 128 * 8; idx += 256) {
      const uint32_t row = idx >> 3, part = idx & 7;
      if (row >= rows) continue;
      uint32_t pi, ip;
      split_token(hd, pos0 + row, &pi, &ip);
      const int32_t page = page_tables[rq.page_table_off + pi];
      if (page < 0 || static_cast<uint32_t>(page) >= kv.n_pages) {
        if (part == 0) atomicAdd(&kv.counters[ctr_index(kCtrBadPages)], 1ull);
        continue;
      }
      *reinterpret_cast<uint4*>(kv.base + static_cast<uint64_t>(page) * kv.page_size + koff + (static_cast<uint64_t>(ip) * 64 + part * 8) * 2) =
          *reinterpret_cast<const uint4*>(&As[row][part * 8]);
    }
    return;
  }
  // V block, stored transposed [d_h][token]: a thread takes one d_h row and 8 consecutive tokens
  const uint64_t voff = kv_block_offset(hd, layer, 1, head, 2);
  for (uint32_t idx = tid; idx < 64 * 16; idx += 256) {
    const uint32_t dh = idx >> 4, t0 = (idx & 15) * 8;
    if (t0 >= rows) continue;
    uint32_t pi, ip;
    split_token(hd, pos0 + t0, &pi, &ip);
    const bool whole = t0 + 8 <= rows && (ip & 7) == 0;  // the 8 tokens are one aligned run inside a page
    if (whole) {
      const int32_t page = page_tables[rq.page_table_off + pi];
      if (page < 0 || static_cast<uint32_t>(page) >= kv.n_pages) {
        if (dh == 0) atomicAdd(&kv.counters[ctr_index(kCtrBadPages)], 1ull);
        continue;
      }
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = As[t0 + 2 * e][dh] | (static_cast<uint32_t>(As[t0 + 2 * e + 1][dh]) << 16);
      *reinterpret_cast<uint4*>(kv.base + static_cast<uint64_t>(page) * kv.page_size + voff + (static_cast<uint64_t>(dh) * hd.pt + ip) * 2) =
          make_uint4(w[0], w[1], w[2], w[3]);
    } else {
      for (uint32_t e = 0; e < 8 && t0 + e < rows; ++e) {
        split_token(hd, pos0 + t0 + e, &pi, &ip);
        const int32_t page = page_tables[rq.page_table_off + pi];
        if (page < 0 || static_cast<uint32_t>(page) >= kv.n_pages) {
          if (dh == 0) atomicAdd(&kv.counters[ctr_index(kCtrBadPages)], 1ull);
          continue;
        }
        *reinterpret_cast<uint16_t*>(kv.base + static_cast<uint64_t>(page) * kv.page_size + voff + (static_cast<uint64_t>(dh) * hd.pt + ip) * 2) =
            As[t0 + e][dh];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Fused layer halves for bf16 models of width KD = 64, 128, 256 or 512 (one kernel each, no normalised copy of the
// activations in memory):
//   FRONT: [U|V|Q|K] = SiLU(LN1(X) W1 + b1), U and Q*log2(e) to row-major buffers, K and V into
//          the pages;
//   BACK:  Y = X + (LN2(O) * U) W2 + b2.
// (X, Q, K, V, Y are bf16; O, U, the normalised operand and the weight copies are half precision.)
// A wavefront owns 32 consecutive token rows, whichever requests they belong to.  Their activations are loaded once
// (whole-line loads, dealt out to the lanes through LDS, 64 columns at a time), normalised in registers (a row is split
// over the two lanes (g = 0, 1) that share the token: two cross-lane sums) and kept as the token-side MFMA operand
// for the whole sweep over the output columns, KD/16 fragments of 8 elements.  The weights are stored in the order of
// the MFMA operand (weight_fragments below), so a tile of 32 output columns is one contiguous piece that
// global_load_lds copies into LDS as it is, double buffered, without passing through registers, and an operand read
// is 64 lanes times 16 consecutive bytes.  The product is taken as (W tile) x (X^T), so a
// lane ends up with one token and 16 output features (four runs of four); row-major outputs and
// K rows pass through a wave-private LDS tile and leave as 16-byte stores, V^T leaves as
// lane-coalesced 2-byte stores.
// A tile's weights are fetched while the tile before it is multiplied, and waited for just before that tile's results
// are stored: the wait (which counts loads and stores in issue order) then never covers stores just issued.
// A block sweeps all column tiles when there are rows enough to fill the chip, else the columns are cut too, down to one
// tile a block (the launcher's rule).  Steps with fewer rows take layer_join instead (layers_joined says which).
// What bounds it, d = 256, 131 440 rows: the front half moves 0.39 GB (0.34 of them its rows), and vector (49% of its
// cycles), matrix (30%) and LDS (32%) work lie only partly on top of one another (25% of the time neither of the first two
// runs); the back half moves 0.31 GB at 4.9 TB/s.  Three blocks per CU and the rows in uneven rounds 126 and 68 us, four,
// which 40 KB of LDS and 128 registers allow, 119 to 123 and 61 to 64; 145 000 rows, where the last round was nearly
// empty: 140 -> 126 us and 70 -> 67.  Stores into pages that the compiler knows to be global (it had waited for all LDS reads
// before each pair of products, because a flat store counts as one), packing without a branch per run and fragments read four
// steps ahead: the front half 120 -> 110.5 us in turn (108 to 117 on other cards), a step of 64 histories of 2048 1.3% less, of 32 x 512 at d = 512 1.7%.
// ---------------------------------------------------------------------------------------
struct LayerHalfArgs {
  HstuDims hd;
  uint32_t layer;
  uint32_t n_rows;
  const uint16_t* a_in;    // FRONT: X   BACK: O       [N][KD]
  const uint16_t* gate;    // BACK: U
  const float* ln_g;
  const float* ln_b;
  const uint16_t* wf;      // weight fragments of this layer
  const float* bias;       // [n_out]
  uint16_t* u;             // FRONT outputs
  uint16_t* q;
  KvView kv;
  const ReqDev* reqs;
  const uint32_t* group_req;  // request of row 32 i, and behind the last one the last row's
  const int32_t* page_tables;
  const uint16_t* resid;   // BACK: X
  uint16_t* y;             // BACK output
  // Row tiles [0, rows0) in blocks of cb0 32-column tiles each (one or two column ranges), then rows1 more in blocks of
  // cb1; the ranges of a row tile lie rows0 (rows1) blocks apart, and rows1_inv = 2^31 / rows1, rounded up
  uint32_t rows0, cb0, blocks0, rows1, cb1, rows1_inv;
};

__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
  typedef float v2f __attribute__((ext_vector_type(2)));
  const v2f v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2bf));
}
__device__ __forceinline__ void unpack8(const u32x4& a, float v[8]) {  // eight bf16
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[2 * k] = __uint_as_float(w[k] << 16);
    v[2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
  }
}
__device__ __forceinline__ void unpack8h(const u32x4& a, float v[8]) {  // eight half-precision values
  const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const f16x2 h = __builtin_bit_cast(f16x2, w[k]);
    v[2 * k] = static_cast<float>(h[0]);
    v[2 * k + 1] = static_cast<float>(h[1]);
  }
}
// the rows a layer half normalises: the bf16 residual stream (front) or the half-precision attention output (back)
template <bool FRONT>
__device__ __forceinline__ void unpack_in(const u32x4& a, float v[8]) {
  if (FRONT) unpack8(a, v);
  else unpack8h(a, v);
}

// Tells the compiler nothing about the value it returns: the unpacked fp32 copy of a row that an
// earlier pass over the registers made cannot be kept alive for a later pass (it would double
// the registers the row takes).
__device__ __forceinline__ void forget(u32x4& a) { asm volatile("" : "+v"(a)); }

// Copies 16 bytes per lane from base + voff to the LDS address lds + 16 * lane without passing through registers; lds and
// base are the wavefront's.  The compiler does not know about the copy: the wavefront waits for it with wait_vm, other
// wavefronts see it behind a barrier.  (With the builtin of the same instruction the compiler waits for all outstanding
// copies before every LDS read.)
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)p));
}
__device__ __forceinline__ const uint8_t* in_scalar(const uint8_t* p) {  // a pointer all lanes agree on, in scalar registers
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a)), hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
  return reinterpret_cast<const uint8_t*>((static_cast<uint64_t>(hi) << 32) | lo);
}
// An address in a page.  A pointer that was put together from integers has to be said to be global: stores the compiler takes
// for ones that may go to LDS make it wait for all LDS reads at each use of one.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* in_global(uint8_t* p) { return (__attribute__((address_space(1))) T*)p; }
// (The LDS address goes into m0, which the compiler may use for itself between any two statements: one statement writes it,
// waits and copies.  The instruction needs one wait state behind a write of m0, and five behind a vector instruction,
// v_readfirstlane for one, that has written its scalar base.  The compiler keeps that distance for its own instructions
// but does not look into this one.)
// (m0 is reserved: the compiler holds nothing there across statements unless it sees that nobody writes it, which is what
// the clobber says.  The warning that it will not be saved is beside the point.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int COPIES>  // one KB, or two that follow each other in both places (four in one statement: the back half at d = 256 spills)
__device__ __forceinline__ void copy_to_lds(uint32_t lds, const void* base, uint32_t voff) {
  static_assert(COPIES == 1 || COPIES == 2);
  if constexpr (COPIES == 1)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024"
                 ::"s"(lds), "v"(voff), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void copy_to_lds_from(uint32_t lds, const void* src) {  // from an address of each lane's own
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// f(0), f(1), .. f(N - 1) with constant arguments: unrolled whatever its size, so that the arrays it indexes are registers
template <int... I, typename F>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F f) {
  unrolled(std::make_integer_sequence<int, N>{}, f);
}

constexpr uint32_t kMaxSweep = 1024;  // output columns a block sweeps at most (a layer half has at most twice as many)

template <int KD, bool FRONT, int WPB>
__global__ __launch_bounds__(64 * WPB, KD <= 256 ? 4 : 2) void layer_half_fused(LayerHalfArgs a) {
  constexpr int kSt = KD / 16;        // MFMA steps over the contraction
  constexpr int kPieces = KD / 64;    // 64-column pieces of a row
  constexpr int kTileBytes = kSt * 1024;
  constexpr int kCopies = kSt / WPB;  // 1 KB copies of a weight tile per wavefront
  static_assert(kSt % WPB == 0 && KD % 64 == 0 && (kCopies == 1 || kCopies % 2 == 0), "a weight tile must split evenly over the block");
  constexpr int kStageBytes = WPB * 4096;        // row dealing: 32 rows of 128 bytes per wavefront
  constexpr uint32_t kOutTok = KD == 256 ? 16 : 32;  // tokens in a wavefront's output tile: with all 32 the fourth block would not fit the CU
  constexpr int kOutBytes = WPB * kOutTok * 64;
  constexpr bool kStageInTile = kTileBytes >= kStageBytes;  // the dealing happens in the second weight buffer, else in the output tiles
  __shared__ __attribute__((aligned(16))) uint8_t wtile[2][kTileBytes];
  __shared__ __attribute__((aligned(16))) uint8_t otile[(kStageInTile ? 0 : kStageBytes) > kOutBytes ? kStageBytes : kOutBytes];
  __shared__ __attribute__((aligned(16))) float lnp_own[kStageInTile ? 4 : 2 * KD];
  __shared__ __attribute__((aligned(16))) float bias_s[FRONT ? kMaxSweep : KD];
  // LayerNorm scale and shift: in the output tiles, which the sweep takes over, unless the row dealing is there
  static_assert(!kStageInTile || 2 * KD * 4 <= kOutBytes, "LayerNorm parameters fit the output tiles");
  float* lnp = kStageInTile ? reinterpret_cast<float*>(&otile[0]) : lnp_own;
  const uint32_t tid = threadIdx.x, lane = tid & 63, g = lane >> 5, li = lane & 31;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool rest = blockIdx.x >= a.blocks0;
  const uint32_t bx = rest ? blockIdx.x - a.blocks0 : blockIdx.x;
  const uint32_t col = rest ? static_cast<uint32_t>(static_cast<uint64_t>(bx) * a.rows1_inv >> 31) : (bx >= a.rows0 ? 1 : 0);
  const uint32_t n_cb = rest ? a.cb1 : a.cb0, cb0 = col * n_cb;
  const uint32_t tile = rest ? a.rows0 + bx - col * a.rows1 : bx - col * a.rows0;
  const uint32_t r0 = (tile * WPB + wave) * 32;  // this wavefront's first row
  const HstuDims& hd = a.hd;

  const uint32_t wlds = __builtin_amdgcn_readfirstlane(lds_address(&wtile[0][0])) + wave * (kCopies * 1024);
  auto fetch_w = [&](uint32_t cb, uint32_t buf) {
    const uint8_t* src = reinterpret_cast<const uint8_t*>(a.wf) + static_cast<uint64_t>(cb) * kTileBytes + wave * (kCopies * 1024);
#pragma unroll
    for (int c = 0; c < kCopies; c += 2)
      copy_to_lds<kCopies < 2 ? 1 : 2>(wlds + buf * kTileBytes + c * 1024, src + c * 1024, lane * 16);
  };

  // ---- activation rows: issue the loads ---------------------------------------------------------
  // One load instruction covers 128 bytes of eight rows.  A piece (64 columns of the 32 rows) is dealt out to the
  // operand layout (lane = token, 8 of every 16 elements) through 4 KB of wave-private LDS; chunk c of row r sits at
  // c ^ (r / 2 mod 8), where no two lanes served together meet in a bank.  Rows past the end read the first row; their results are never stored.
  const uint32_t st_r = lane >> 3, st_c = lane & 7;
  auto issue_piece = [&](const uint16_t* src, int p, u32x4 (&v)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t r = r0 + 8 * i + st_r;
      v[i] = *reinterpret_cast<const u32x4*>(src + static_cast<uint64_t>(r < a.n_rows ? r : 0) * KD + 64 * p + 8 * st_c);
    }
  };
  uint8_t* stage = (kStageInTile ? &wtile[1][0] : &otile[0]) + wave * 4096;
  auto deal_piece = [&](const u32x4 (&v)[4], auto& dst, auto at) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t r = 8 * i + st_r;
      *reinterpret_cast<u32x4*>(stage + r * 128 + 16 * (st_c ^ (r >> 1 & 7))) = v[i];
    }
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) dst[at + s2] = *reinterpret_cast<const u32x4*>(stage + li * 128 + 16 * ((2 * s2 + g) ^ (li >> 1 & 7)));
  };
  u32x4 xr[kSt];  // this lane's half of its token's row: raw, then normalised (and gated) half precision
  {
    u32x4 raw[kPieces][4];
    unrolled<kPieces>([&](auto p) { issue_piece(a.a_in, p, raw[p]); });
    fetch_w(cb0, 0);
    unrolled<kPieces>([&](auto p) { deal_piece(raw[p], xr, std::integral_constant<int, 4 * p>{}); });
  }
  // BACK: the gate rows follow, a piece or two ahead of their use (what the registers of the block count above allow)
  constexpr int kGates = KD == 256 ? 1 : kPieces < 2 ? 1 : 2;
  u32x4 gate[kGates][4];
  if constexpr (!FRONT) unrolled<kGates>([&](auto p) { issue_piece(a.gate, p, gate[p]); });
  for (uint32_t i = tid; i < KD; i += 64 * WPB) {
    lnp[i] = a.ln_g[i];
    lnp[KD + i] = a.ln_b[i];
  }
  for (uint32_t i = tid; i < n_cb * 32; i += 64 * WPB) bias_s[i] = a.bias[cb0 * 32 + i];

  // ---- where this lane's token goes (these dependent loads fly during the LayerNorm) ----------------
  const bool row_ok = r0 + li < a.n_rows;
  const uint8_t* page_ptr = nullptr;  // FRONT: start of the token's page (nullptr: no such row, or a bad page id)
  uint32_t tok = 0;
  if (FRONT && row_ok) {
    const uint32_t row = r0 + li, grp = r0 / 32;
    const ReqDev rq = a.reqs[request_of(a.reqs, row, a.group_req[grp], a.group_req[grp + 1])];
    uint32_t pi;
    split_token(hd, rq.prefix_len + (row - rq.x_off), &pi, &tok);
    const int32_t page = a.page_tables[rq.page_table_off + pi];
    if (page < 0 || static_cast<uint32_t>(page) >= a.kv.n_pages) {
      if (col == 0 && g == 0) atomicAdd(&a.kv.counters[ctr_index(kCtrBadPages)], 1ull);
    } else {
      page_ptr = a.kv.base + static_cast<uint64_t>(page) * a.kv.page_size;
    }
  }

  // ---- normalise, keep as MFMA operand -----------------------------------------------------------
  {
    float s = 0.0f;
    unrolled<kSt>([&](auto st) {
      float v[8];
      unpack_in<FRONT>(xr[st], v);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[e];
    });
    s += __shfl_xor(s, 32, 64);
    const float mean = s / KD;
    float qq = 0.0f;
    unrolled<kSt>([&](auto st) { forget(xr[st]); });
    unrolled<kSt>([&](auto st) {
      float v[8];
      unpack_in<FRONT>(xr[st], v);
#pragma unroll
      for (int e = 0; e < 8; ++e) qq += (v[e] - mean) * (v[e] - mean);
    });
    qq += __shfl_xor(qq, 32, 64);
    const float rstd = 1.0f / sqrtf(qq / KD + hd.eps);
    __syncthreads();  // lnp is visible
    unrolled<kSt>([&](auto st) { forget(xr[st]); });
    unrolled<kPieces>([&](auto p) {
      u32x4 gr[4];
      if constexpr (!FRONT) {
        deal_piece(gate[p % kGates], gr, std::integral_constant<int, 0>{});
        if (p + kGates < kPieces) issue_piece(a.gate, p + kGates, gate[p % kGates]);
      }
      unrolled<4>([&](auto s2) {
        constexpr int st = 4 * p + s2;
        float v[8], gg[8], bb[8];
        unpack_in<FRONT>(xr[st], v);
        load8(lnp + 16 * st + 8 * g, gg);
        load8(lnp + KD + 16 * st + 8 * g, bb);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (v[e] - mean) * rstd * gg[e] + bb[e];
        if constexpr (!FRONT) {
          float uv[8];
          unpack8h(gr[s2], uv);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] *= uv[e];
        }
        xr[st] = u32x4{pack2_f16(v[0], v[1]), pack2_f16(v[2], v[3]), pack2_f16(v[4], v[5]), pack2_f16(v[6], v[7])};
        // the result is pinned down here and memory operations may not pass: the LDS reads of later
        // steps stay behind this step's arithmetic instead of piling up in registers
        forget(xr[st]);
        asm volatile("" ::: "memory");
      });
    });
  }

  // Row-major outputs leave through a wave-private LDS tile that turns "one token, four runs of four features per lane"
  // into 16-byte pieces, kOutTok tokens at a time: lane l stores features 8 (l % 4) .. + 8 of tokens l / 4 and l / 4 + 16,
  // so four lanes cover 64 contiguous bytes of a row (32 bytes: 4% slower).  Chunk c of row r sits at c ^ (r / 4 mod 4),
  // so that the rows' 64 bytes cover all banks.
  const uint32_t st_row = lane >> 2, st_col = lane & 3;
  const bool st_ok[2] = {r0 + st_row < a.n_rows, r0 + st_row + 16 < a.n_rows};
  const uint64_t st_off = static_cast<uint64_t>(r0 + st_row) * KD + 8 * st_col;
  uint8_t* kdst[2] = {nullptr, nullptr};  // FRONT: this lane's 16 bytes of the tokens' K rows inside their pages, before the head's offset
  if (FRONT) {
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const uint64_t own = reinterpret_cast<uint64_t>(page_ptr);
      const uint32_t rl = st_row + 16 * h2;
      const uint32_t lo = __shfl(static_cast<uint32_t>(own), rl, 64), hi = __shfl(static_cast<uint32_t>(own >> 32), rl, 64);
      const uint32_t tk = __shfl(tok, rl, 64);
      const uint64_t pp = (static_cast<uint64_t>(hi) << 32) | lo;
      if (pp) kdst[h2] = reinterpret_cast<uint8_t*>(pp) + tk * 128 + 16 * st_col;
    }
  }
  uint8_t* ot = &otile[0] + wave * (kOutTok * 64);
  auto transposed = [&](const u32x2 (&run)[4], u32x4 (&v)[2]) {  // run[k]: this lane's features 8 k + 4 g .. + 4 of its token
#pragma unroll
    for (uint32_t h2 = 0; h2 < 2; ++h2) {
      if (kOutTok == 32 ? h2 == 0 : li >> 4 == h2) {
#pragma unroll
        for (uint32_t r4 = 0; r4 < 4; ++r4)
          *reinterpret_cast<u32x2*>(ot + (li % kOutTok) * 64 + 16 * (r4 ^ ((li >> 2) & 3)) + 8 * g) = run[r4];
      }
      v[h2] = *reinterpret_cast<const u32x4*>(ot + (st_row + (kOutTok - 16) * h2) * 64 + 16 * (st_col ^ ((st_row >> 2) & 3)));
      asm volatile("" : "+v"(v[h2]));  // all lanes have read before any lane goes on to write the next part
    }
  };

  // ---- sweep over the output columns ----------------------------------------------------------
  const uint64_t own_off = static_cast<uint64_t>(row_ok ? r0 + li : 0) * KD + 4 * g;  // BACK: the lane's first residual run
  wait_vm<0>();
  for (uint32_t k = 0; k < n_cb; ++k) {
    const uint32_t cb = cb0 + k, n0 = cb * 32;
    __syncthreads();  // tile k is in LDS, and every wavefront is done with tile k - 1, whose buffer takes tile k + 1
    if (k + 1 < n_cb) fetch_w(cb + 1, (k + 1) & 1);
    if (r0 >= a.n_rows) {  // a wavefront without rows only helps to fetch
      wait_vm<0>();
      continue;
    }
    u32x2 res[4];  // BACK: the residual of this lane's token, four runs of four features
    if (!FRONT) {
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) res[r4] = *reinterpret_cast<const u32x2*>(a.resid + own_off + n0 + 8 * r4);
    }
    f32x16 acc;
    // acc[e]: feature n0 + 8*(e/4) + 4*g + e%4 of this lane's token; the bias is the starting value
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 b = *reinterpret_cast<const float4*>(bias_s + k * 32 + 8 * r4 + 4 * g);
      acc[4 * r4] = b.x; acc[4 * r4 + 1] = b.y; acc[4 * r4 + 2] = b.z; acc[4 * r4 + 3] = b.w;
    }
    const uint8_t* wb = wtile[k & 1] + lane * 16;
#pragma unroll
    for (int st = 0; st < kSt; ++st) {
      const f16x8 wf = __builtin_bit_cast(f16x8, *reinterpret_cast<const u32x4*>(wb + st * 1024));
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf, __builtin_bit_cast(f16x8, xr[st]), acc, 0, 0, 0);
    }
    // Fragments are read four steps ahead (the bias and four, then one per product, 0x100: LDS reads, 0x8: MFMA); left to itself the
    // compiler reads two, uses both and reads the next two.
    if constexpr (kSt > 4) {
      __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);
      unrolled<kSt - 4>([&](auto) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      });
      __builtin_amdgcn_sched_group_barrier(0x8, 4, 0);
    }
    if (FRONT) {
      const uint32_t which = n0 / KD, c0 = n0 % KD;  // 0: U, 1: V, 2: Q, 3: K
      float z[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) z[e] = acc[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-acc[e]));
      if (which == 1) {
        wait_vm<0>();
        // V block [64][page_tokens]: the 32 lanes of a half-wave write 32 consecutive tokens of one feature
        if (page_ptr) {
          const uint32_t head = c0 / 64, cc = c0 % 64 + 4 * g;
          uint8_t* dst = const_cast<uint8_t*>(page_ptr) + kv_block_offset(hd, a.layer, 1, head, 2) + 2 * (static_cast<uint64_t>(cc) * hd.pt + tok);
#pragma unroll
          for (int e = 0; e < 16; e += 2) {
            const uint32_t two = pack2_bf16(z[e], z[e + 1]);
            *in_global<uint16_t>(dst + 2 * static_cast<uint64_t>(8 * (e / 4) + e % 4) * hd.pt) = static_cast<uint16_t>(two);
            *in_global<uint16_t>(dst + 2 * static_cast<uint64_t>(8 * (e / 4) + e % 4 + 1) * hd.pt) = static_cast<uint16_t>(two >> 16);
          }
        }
        continue;
      }
      u32x2 run[4];
      if (which == 0) {  // U is the library's own (half precision); Q and K are bf16
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) run[r4] = u32x2{pack2_f16(z[4 * r4], z[4 * r4 + 1]), pack2_f16(z[4 * r4 + 2], z[4 * r4 + 3])};
      } else {
        if (which == 2) {  // the attention kernel wants q * log2(e)
#pragma unroll
          for (int e = 0; e < 16; ++e) z[e] *= 1.4426950408889634f;
        }
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) run[r4] = u32x2{pack2_bf16(z[4 * r4], z[4 * r4 + 1]), pack2_bf16(z[4 * r4 + 2], z[4 * r4 + 3])};
      }
      u32x4 v[2];
      transposed(run, v);
      wait_vm<0>();
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        if (which == 3) {  // K block [token][64]
          if (kdst[h2]) *in_global<u32x4>(kdst[h2] + kv_block_offset(hd, a.layer, 0, c0 / 64, 2) + (c0 % 64) * 2) = v[h2];
        } else if (st_ok[h2]) {
          *reinterpret_cast<u32x4*>((which == 0 ? a.u : a.q) + st_off + 16 * KD * h2 + c0) = v[h2];
        }
      }
    } else {
      u32x2 run[4];
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t w = res[r4][e >> 1];
          y[e] = __uint_as_float(e & 1 ? w & 0xFFFF0000u : w << 16) + acc[4 * r4 + e];
        }
        run[r4] = u32x2{pack2_bf16(y[0], y[1]), pack2_bf16(y[2], y[3])};
      }
      u32x4 v[2];
      transposed(run, v);
      wait_vm<0>();
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2)
        if (st_ok[h2]) *reinterpret_cast<u32x4*>(a.y + st_off + 16 * KD * h2 + n0) = v[h2];
    }
  }
}

// ---------------------------------------------------------------------------------------
// Small steps, whose kernels are chains of a few dependent round trips: the back half of a layer and the front half of the
// next one in one kernel (both work on rows alone), or either of them alone at the ends of a step.
// A block takes 32 rows and a slice of the front half's columns.  It computes the whole back half of its rows (each
// slice again: a few hundred MFMA cycles) and keeps the layer's output, as bf16 like the matrix it also stores, in LDS.
// The four wavefronts normalise eight rows each, lanes along the rows, and leave the operand in LDS; in the products they
// have output columns of their own, so that weight fragments go from memory straight into registers, a tile ahead, and
// nothing is staged.  What bounds it: about six dependent steps (rows, LayerNorm, product, LayerNorm, product, stores), so
// nothing that a step needs is asked for only there: parameters, biases and the residual come with the rows, a row's page is on
// its way during the back half (64 rows of d = 256 9.2 -> 8.2 us a kernel, 8192 rows 27.9 -> 25.6, 2470 of d = 128 9.9 -> 8.7).
// Steps of four layers with the halves in kernels of their own and joined: 64 rows of d = 256 88 -> 65 us, 8192 rows
// 154 -> 135; 2470 rows of d = 128 97 -> 84; 1024 rows of d = 64 63 -> 51, of d = 512 148 -> 120.
// ---------------------------------------------------------------------------------------
struct JoinArgs {
  HstuDims hd;
  uint32_t layer;          // of the front half
  uint32_t n_rows, groups, front_tiles;  // row groups of 32; column tiles of the front half per wavefront
  // back half
  const uint16_t* o;
  const uint16_t* gate;
  const float* ln2_g;
  const float* ln2_b;
  const uint16_t* w2f;
  const float* b2;
  uint16_t* y;
  // front half
  const float* ln1_g;
  const float* ln1_b;
  const uint16_t* w1f;
  const float* b1;
  uint16_t* u;
  uint16_t* q;
  KvView kv;
  const ReqDev* reqs;
  const uint32_t* group_req;
  const int32_t* page_tables;
  const uint16_t* x;       // the back half's residual, or (alone) what the front half takes
};

template <int KD, bool BACK, bool FRONT>
__device__ __forceinline__ void layer_join_block(JoinArgs a, const ReqDev* reqs, const uint32_t* group_req) {
  constexpr int kSt = KD / 16;       // MFMA steps over the contraction
  constexpr int kOwn = KD / 64;      // 16-byte pieces of a row per lane, eight lanes along a row
  constexpr uint32_t kRowBytes = KD * 2;
  __shared__ __attribute__((aligned(16))) uint8_t operand[32 * kRowBytes];
  __shared__ __attribute__((aligned(16))) uint8_t rows[BACK ? 32 * kRowBytes : 16];
  __shared__ __attribute__((aligned(16))) uint8_t otile[FRONT ? 4 * 2048 : 16];
  // LayerNorm scales and shifts and biases: [ln2_g | ln2_b | b2] and [ln1_g | ln1_b | b1, the slice's columns]
  constexpr int kBackPar = BACK ? 3 * KD : 0;
  __shared__ __attribute__((aligned(16))) float par[kBackPar + (FRONT ? 6 * KD : 0)];
  const uint32_t tid = threadIdx.x, lane = tid & 63, g = lane >> 5, li = lane & 31;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t slice = blockIdx.x / a.groups, group = blockIdx.x - slice * a.groups, r0 = group * 32;
  const HstuDims& hd = a.hd;
  // piece c of row r sits at c ^ swizzle: the operand reads (a row per lane) of lanes that are served together meet in no bank
  auto at = [](uint32_t r, uint32_t c) { return r * kRowBytes + 16 * (c ^ (KD >= 128 ? r & 15 : r >> 1 & 7)); };
  const uint32_t own_r = 8 * wave + (lane >> 3), own_c = lane & 7;  // this lane's pieces: own_c + 8 k of row own_r
  const bool own_ok = r0 + own_r < a.n_rows;
  const uint64_t own_off = static_cast<uint64_t>(own_ok ? r0 + own_r : 0) * KD + 8 * own_c;
  auto load_own = [&](const uint16_t* m, u32x4 (&v)[kOwn]) {
#pragma unroll
    for (int k = 0; k < kOwn; ++k) v[k] = *reinterpret_cast<const u32x4*>(m + own_off + 64 * k);
  };
  // weight fragments of a column tile
  u32x4 w[kSt];
  auto load_w = [&](const uint16_t* wf, uint32_t cb, int st) {
    return *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(wf) + static_cast<uint64_t>(cb) * (kSt * 1024) + st * 1024 + lane * 16);
  };
  const uint32_t front0 = FRONT ? (slice * 4 + wave) * a.front_tiles : 0;  // this wavefront's first column tile of the front half
  const bool has_back = BACK && wave < KD / 32;
  // Everything whose address is known goes out at once: what the first LayerNorm needs, the parameters of all that follows, the
  // residual, the first weights.  The parameters go to LDS, a word or a few per thread, and the residual into the tile of output
  // rows, where each lane finds its part and puts the result in its place.
  u32x4 v[kOwn];
  load_own(BACK ? a.o : a.x, v);
  u32x4 gt[BACK ? kOwn : 1], res[BACK ? kOwn : 1];
  if constexpr (BACK) load_own(a.gate, gt);
  constexpr int kPar = (KD + 255) / 256, kB1 = FRONT ? (4 * KD + 255) / 256 : 1;  // words per thread: of an array of KD, of b1
  const uint32_t b1_n = FRONT ? a.front_tiles * 128 : 0, b1_0 = slice * b1_n;
  float pb[BACK ? 3 * kPar : 1], pf[FRONT ? 2 * kPar : 1], p1[kB1];
  auto par_words = [&](auto f) {  // f(word of the thread, where it lies in an array of KD)
#pragma unroll
    for (int j = 0; j < kPar; ++j)
      if (KD % 256 == 0 || tid < KD) f(j, tid + 256 * j);
  };
  auto b1_words = [&](auto f) {
#pragma unroll
    for (int j = 0; j < kB1; ++j)
      if (tid + 256 * j < b1_n) f(j, tid + 256 * j);
  };
  par_words([&](int j, uint32_t i) {
    if constexpr (BACK) {
      pb[3 * j] = a.ln2_g[i];
      pb[3 * j + 1] = a.ln2_b[i];
      pb[3 * j + 2] = a.b2[i];
    }
    if constexpr (FRONT) {
      pf[2 * j] = a.ln1_g[i];
      pf[2 * j + 1] = a.ln1_b[i];
    }
  });
  if constexpr (FRONT) b1_words([&](int j, uint32_t i) { p1[j] = a.b1[b1_0 + i]; });
  if constexpr (BACK) load_own(a.x, res);
  if (BACK && has_back) unrolled<kSt>([&](auto st) { w[st] = load_w(a.w2f, wave, st); });
  if (FRONT && !BACK) unrolled<kSt>([&](auto st) { w[st] = load_w(a.w1f, front0, st); });

  // ---- FRONT: where this lane's token goes -------------------------------------------------------------------------
  // (The request through scalar loads where the group's rows are of two requests at most, so that it is not waited for behind the
  // loads above; the page's number is looked at when the front half begins.)
  const bool row_ok = r0 + li < a.n_rows;
  int32_t page = -1;
  uint32_t tok = 0;
  if constexpr (FRONT) {
    const uint32_t row = row_ok ? r0 + li : a.n_rows - 1;
    const uint32_t lo = group_req[group], hi = group_req[group + 1];
    uint32_t first, table;  // of the row's request: the token that its row 0 would be, and its page table
    if (hi - lo <= 1) {
      auto word = [](uint32_t x) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(x)); };
      const uint32_t first0 = word(reqs[lo].prefix_len - reqs[lo].x_off), table0 = word(reqs[lo].page_table_off);
      const uint32_t first1 = word(reqs[hi].prefix_len - reqs[hi].x_off), table1 = word(reqs[hi].page_table_off);
      const bool second = word(reqs[hi].x_off) <= row;
      first = second ? first1 : first0;
      table = second ? table1 : table0;
    } else {
      const ReqDev rq = reqs[request_of(reqs, row, lo, hi)];
      first = rq.prefix_len - rq.x_off;
      table = rq.page_table_off;
      asm volatile("" : "+v"(first), "+v"(table));  // (waited for here and not where the two ways meet)
    }
    uint32_t pi;
    split_token(hd, first + row, &pi, &tok);
    page = a.page_tables[table + pi];
  }

  // LayerNorm of row own_r (two passes in fp32, over the eight lanes that share it), times the gate, into the operand
  auto normalise = [&](auto first, const float* ln_g, const float* ln_b, auto ready) {  // ready(): the parameters are in LDS
    constexpr bool kFirst = decltype(first)::value;  // of the front half: bf16 rows, no gate
    float s = 0.0f;
    unrolled<kOwn>([&](auto k) {
      float x[8];
      unpack_in<kFirst>(v[k], x);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += x[e];
    });
    const float mean = group_sum<8>(s) / KD;
    float qq = 0.0f;
    unrolled<kOwn>([&](auto k) {
      float x[8];
      unpack_in<kFirst>(v[k], x);
#pragma unroll
      for (int e = 0; e < 8; ++e) qq += (x[e] - mean) * (x[e] - mean);
    });
    const float rstd = 1.0f / sqrtf(group_sum<8>(qq) / KD + hd.eps);
    ready();
    unrolled<kOwn>([&](auto k) {
      float x[8], gg[8], bb[8];
      unpack_in<kFirst>(v[k], x);
      load8(ln_g + 8 * own_c + 64 * k, gg);
      load8(ln_b + 8 * own_c + 64 * k, bb);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = (x[e] - mean) * rstd * gg[e] + bb[e];
      if constexpr (!kFirst) {
        float uv[8];
        unpack8h(gt[k], uv);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] *= uv[e];
      }
      *reinterpret_cast<u32x4*>(operand + at(own_r, own_c + 8 * k)) =
          u32x4{pack2_f16(x[0], x[1]), pack2_f16(x[2], x[3]), pack2_f16(x[4], x[5]), pack2_f16(x[6], x[7])};
    });
  };
  u32x4 xr[kSt];  // the token-side operand: lane (g, li) holds elements 16 st + 8 g .. + 8 of row li
  auto read_operand = [&]() {
    unrolled<kSt>([&](auto st) { xr[st] = *reinterpret_cast<const u32x4*>(operand + at(li, 2 * st + g)); });
  };
  // acc[e]: column 8 (e / 4) + 4 g + e % 4 of a tile of this lane's token, on top of the tile's bias; the registers of the
  // weights take the next tile's as they become free
  auto product = [&](const float* bias, auto next, const uint16_t* next_w, uint32_t next_cb) {
    f32x16 acc;
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 b = *reinterpret_cast<const float4*>(bias + 8 * r4 + 4 * g);
      acc[4 * r4] = b.x; acc[4 * r4 + 1] = b.y; acc[4 * r4 + 2] = b.z; acc[4 * r4 + 3] = b.w;
    }
    unrolled<kSt>([&](auto st) {
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w[st]), __builtin_bit_cast(f16x8, xr[st]), acc, 0, 0, 0);
      if constexpr (decltype(next)::value) w[st] = load_w(next_w, next_cb, st);
    });
    return acc;
  };

  // the parameters and the residual go to LDS before the first LayerNorm's second part
  auto put_par = [&]() {
    par_words([&](int j, uint32_t i) {
      if constexpr (BACK) {
        par[i] = pb[3 * j];
        par[KD + i] = pb[3 * j + 1];
        par[2 * KD + i] = pb[3 * j + 2];
      }
      if constexpr (FRONT) {
        par[kBackPar + i] = pf[2 * j];
        par[kBackPar + KD + i] = pf[2 * j + 1];
      }
    });
    if constexpr (FRONT) b1_words([&](int j, uint32_t i) { par[kBackPar + 2 * KD + i] = p1[j]; });
    if constexpr (BACK) unrolled<kOwn>([&](auto k) { *reinterpret_cast<u32x4*>(rows + at(own_r, own_c + 8 * k)) = res[k]; });
    __syncthreads();
  };
  if constexpr (BACK) {
    normalise(std::false_type{}, par, par + KD, put_par);
    __syncthreads();
    read_operand();
    for (uint32_t cb = wave; cb < KD / 32; cb += 4) {
      const bool last = cb + 4 >= KD / 32;
      f32x16 acc;
      if (FRONT) acc = product(par + 2 * KD + 32 * cb, std::true_type{}, last ? a.w1f : a.w2f, last ? front0 : cb + 4);
      else if (last) acc = product(par + 2 * KD + 32 * cb, std::false_type{}, nullptr, 0);
      else acc = product(par + 2 * KD + 32 * cb, std::true_type{}, a.w2f, cb + 4);
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        u32x2* run = reinterpret_cast<u32x2*>(rows + at(li, 4 * cb + r4) + 8 * g);  // four columns of this lane's token
        const u32x2 before = *run;
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t x = before[e >> 1];
          y[e] = __uint_as_float(e & 1 ? x & 0xFFFF0000u : x << 16) + acc[4 * r4 + e];
        }
        *run = u32x2{pack2_bf16(y[0], y[1]), pack2_bf16(y[2], y[3])};
      }
    }
    if (FRONT && !has_back) unrolled<kSt>([&](auto st) { w[st] = load_w(a.w1f, front0, st); });
    __syncthreads();
    unrolled<kOwn>([&](auto k) { v[k] = *reinterpret_cast<const u32x4*>(rows + at(own_r, own_c + 8 * k)); });
    if (slice == 0 && own_ok) unrolled<kOwn>([&](auto k) { *reinterpret_cast<u32x4*>(a.y + own_off + 64 * k) = v[k]; });
  }
  if constexpr (FRONT) {
    if constexpr (BACK) normalise(std::true_type{}, par + kBackPar, par + kBackPar + KD, []() {});
    else normalise(std::true_type{}, par + kBackPar, par + kBackPar + KD, put_par);
    __syncthreads();
    read_operand();
    const uint8_t* page_ptr = nullptr;
    if (page < 0 || static_cast<uint32_t>(page) >= a.kv.n_pages) {
      if (row_ok && slice == 0 && wave == 0 && g == 0) atomicAdd(&a.kv.counters[ctr_index(kCtrBadPages)], 1ull);
    } else if (row_ok) {
      page_ptr = a.kv.base + static_cast<uint64_t>(page) * a.kv.page_size;
    }
    // stores as in the large kernel: row-major outputs turned into 16-byte pieces in wave-private LDS, V^T by lanes
    const uint32_t st_row = lane >> 2, st_col = lane & 3;
    const bool st_ok[2] = {r0 + st_row < a.n_rows, r0 + st_row + 16 < a.n_rows};
    const uint64_t st_off = static_cast<uint64_t>(r0 + st_row) * KD + 8 * st_col;
    uint8_t* kdst[2] = {nullptr, nullptr};
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const uint64_t own = reinterpret_cast<uint64_t>(page_ptr);
      const uint32_t rl = st_row + 16 * h2;
      const uint32_t lo = __shfl(static_cast<uint32_t>(own), rl, 64), hi = __shfl(static_cast<uint32_t>(own >> 32), rl, 64);
      const uint32_t tk = __shfl(tok, rl, 64);
      const uint64_t pp = (static_cast<uint64_t>(hi) << 32) | lo;
      if (pp) kdst[h2] = reinterpret_cast<uint8_t*>(pp) + tk * 128 + 16 * st_col;
    }
    uint8_t* ot = &otile[0] + wave * 2048;
    for (uint32_t t = 0; t < a.front_tiles; ++t) {
      const uint32_t cb = front0 + t, n0 = cb * 32;
      f32x16 acc;
      if (t + 1 < a.front_tiles) acc = product(par + kBackPar + 2 * KD + n0 - b1_0, std::true_type{}, a.w1f, cb + 1);
      else acc = product(par + kBackPar + 2 * KD + n0 - b1_0, std::false_type{}, nullptr, 0);
      const uint32_t which = n0 / KD, c0 = n0 % KD;  // 0: U, 1: V, 2: Q, 3: K
      float z[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) z[e] = acc[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-acc[e]));
      if (which == 1) {
        if (page_ptr) {
          const uint32_t head = c0 / 64, cc = c0 % 64 + 4 * g;
          uint8_t* dst = const_cast<uint8_t*>(page_ptr) + kv_block_offset(hd, a.layer, 1, head, 2) + 2 * (static_cast<uint64_t>(cc) * hd.pt + tok);
#pragma unroll
          for (int e = 0; e < 16; e += 2) {
            const uint32_t two = pack2_bf16(z[e], z[e + 1]);
            *in_global<uint16_t>(dst + 2 * static_cast<uint64_t>(8 * (e / 4) + e % 4) * hd.pt) = static_cast<uint16_t>(two);
            *in_global<uint16_t>(dst + 2 * static_cast<uint64_t>(8 * (e / 4) + e % 4 + 1) * hd.pt) = static_cast<uint16_t>(two >> 16);
          }
        }
        continue;
      }
      const float sc = which == 2 ? 1.4426950408889634f : 1.0f;
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        *reinterpret_cast<u32x2*>(ot + li * 64 + 16 * (r4 ^ ((li >> 2) & 3)) + 8 * g) =
            which == 0 ? u32x2{pack2_f16(z[4 * r4], z[4 * r4 + 1]), pack2_f16(z[4 * r4 + 2], z[4 * r4 + 3])}
                       : u32x2{pack2_bf16(z[4 * r4] * sc, z[4 * r4 + 1] * sc), pack2_bf16(z[4 * r4 + 2] * sc, z[4 * r4 + 3] * sc)};
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        const u32x4 o16 = *reinterpret_cast<const u32x4*>(ot + (st_row + 16 * h2) * 64 + 16 * (st_col ^ ((st_row >> 2) & 3)));
        if (which == 3) {
          if (kdst[h2]) *in_global<u32x4>(kdst[h2] + kv_block_offset(hd, a.layer, 0, c0 / 64, 2) + (c0 % 64) * 2) = o16;
        } else if (st_ok[h2]) {
          *reinterpret_cast<u32x4*>((which == 0 ? a.u : a.q) + st_off + 16 * KD * h2 + c0) = o16;
        }
      }
      __builtin_amdgcn_wave_barrier();  // the tile is read before the next one is written
    }
  }
}

template <int KD, bool BACK, bool FRONT>
__global__ __launch_bounds__(256, KD <= 256 ? 2 : 1) void layer_join(JoinArgs a) {
  layer_join_block<KD, BACK, FRONT>(a, a.reqs, a.group_req);
}

// ---------------------------------------------------------------------------------------
// bf16 paged attention on MFMA, d_h = 64.  A block of four wavefronts owns 128 consecutive
// queries of one request and one head (32 per wavefront) and walks
// a range of key tiles (64 keys), K [key][d_h] and V^T [d_h][key] of the tile in
// LDS, copied there through the page table while the tile before it is used.
// Each wavefront computes S^T = K Q^T (keys x queries, so a lane ends up holding one query
// and 16 keys), applies bias, SiLU and the causal mask in registers, and feeds the bf16
// result straight back as the second operand of O^T += V^T P^T: the accumulator layout of
// the first product is the operand layout of the second, so the scores never leave
// registers.  K rows are kept in LDS in a permuted order (bits 2 and 3 of the key
// index swapped) so that the 8 keys a lane holds per contraction step are consecutive
// and the matching V^T operand is one 16-byte LDS read.
//
// The epilogue is the binding unit (16 scores per lane against 8 MFMAs), so it is pared
// down to the minimum:
//   - Q arrives multiplied by log2(e) and both bias tables are scaled likewise, so that
//     y = x*log2(e) comes out of the matrix product and SiLU(x) = ln2 * y / (1 + 2^-y);
//     ln2 and 1/n are applied once to the output accumulators;
//   - the positional bias is Toeplitz: the window of the (reversed, scaled) table that a key
//     tile needs sits in LDS, in four copies shifted by one element each so that every lane
//     can read its 8 consecutive entries as aligned 16-byte words, and initialises the score
//     accumulators, so adding it costs no arithmetic; from one tile to the next the window moves by 64 entries,
//     which replace the oldest ones of a ring;
//   - time gaps are taken from 32-bit timestamps relative to the request's first one; for a
//     32x32 block whose smallest and largest gap fall into the same log2 bucket (most blocks
//     away from the diagonal) the time bias is one scalar; if they fall into adjacent
//     buckets it is a compare-and-select per score; other blocks take the bucket per score;
//     requests spanning >= 2^31 s (or models with more than 32 buckets) use 64-bit gaps;
//   - the causal select is applied only in blocks that touch the diagonal.
//
// What the vector unit has to do is fixed by that (633 of its cycles per 32x32 block, 256 of the matrix unit), so
// the rest is to keep it fed: the copies to LDS pass through no registers, which leaves the 128 that four wavefronts
// per SIMD allow, and the block needs 40 KB of LDS, so that four are resident per CU.  With tiles staged through registers
// (168 of them, 48 KB, three per SIMD) a launch over 195M (query, key) pairs, d = 256, took 0.382 ms, so 0.335; over 32 x 512
// queries behind 16 384 keys, d = 512, 0.971 ms, so 0.88.  By the counters the vector unit is busy 74% of the time (55% before),
// one of the two units 88% (68%).
// Behind that came what a launch loses at its end and to LDS banks: the order of the work lists with wavefronts that take
// turns at going first (64 users back with 64 tokens behind 2048 and 64 new histories 0.424 -> 0.355 ms, the d = 512 launch
// 0.881 -> 0.833), and rows laid out for how 16-byte reads are served (0.332 -> 0.324, 0.827 -> 0.817).  On one card the
// first of these launches then ran at 617 TFLOP/s, the second at 683 (cards differ by up to 6%).  By the counters no LDS read
// meets another in a bank.
// A third of the vector instructions beside the epilogue were addresses: of the page (now in scalar registers, its number read a
// tile ahead), of the staged operands (now constants of two copies of the loop's body), of the next window entries; and
// conditions that were kept in vector registers.  Without them, with the next tile's copies between the two halves instead of in
// front of them (128 users back with 64 tokens behind 3072 530 -> 521 us a step) and with
// the first two tiles on their way together, a block takes 823 SIMD cycles (886) and steps take 3 to 5% less: 64 histories of 2048 2044 -> 1975 us, 32 x 512 behind
// 16 384 7.40 -> 7.12 ms, the 128 users 545 -> 520, one of them 102.2 -> 99.3, 13 ragged prefills 103.1 -> 99.
// Measured on it, timing only: without the reciprocal 8% of the d = 512 step, without SiLU and bias 28%, one-bucket bias
// everywhere 1 to 4%.  Kept out, each slower: four copies of the body (by 1%), the last block's bucket remembered (by 2%).
// The 128 registers are too few by five: 20 bytes of scratch a lane, stored once in front of the loop and reloaded behind it.
// ---------------------------------------------------------------------------------------
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr uint32_t kAttnQ = 128;     // queries per block
constexpr uint32_t kPosRing = 256;   // a tile needs 191 distances, the next one 64 new ones
constexpr uint32_t kPosMirror = 24;  // the first entries once more behind the end: a lane reads up to 24 from its first
constexpr uint32_t kPosCopy = 304;   // (the two, and what spreads the copies over the banks)

struct AttnShared {
  // Two staged key tiles: K [key][d_h] and V^T [d_h][key], 64 rows of 128 bytes each.  A 16-byte read is served for sixteen
  // lanes at a time, {0-3, 12-15, 20-27} and {4-11, 16-19, 28-31} of either half wavefront, over 64 banks: chunk c (16
  // bytes) of row r sits at c ^ (r / 2 mod 8), where the operand reads of such lanes (a row each) meet in no bank.
  uint8_t kv[2][2][8192];
  // Copy s holds entry x of the positional window at (x - s) mod kPosRing, so that any 8 consecutive entries can be
  // read as aligned 16-byte words of one of the copies.  The copies lie 192 bytes (mod 256) apart: no bank is met twice
  // here either.
  float pos[4][kPosCopy];
  uint32_t tk[2][64];  // key timestamps of the staged tiles relative to the request's first one
  float time[64];
  float rtime[32];     // rtime[c] = time bias of a gap with c leading zero bits (32-bit gaps, n_time <= 32)
  int32_t pages[kAttnMaxItemPages];  // page ids of the item's key range (-1: outside the pool); the last entry is never one: -1
};
static_assert(sizeof(AttnShared) <= 40960, "four blocks per CU");

__device__ const uint4 kZeroChunk = {0, 0, 0, 0};  // what keys without a page are copied from

__device__ __forceinline__ uint32_t bucket_u32(uint32_t dt, uint32_t n_time) {
  const uint32_t b = dt > 1 ? 31u - static_cast<uint32_t>(__clz(static_cast<int>(dt))) : 0u;
  return b < n_time - 1 ? b : n_time - 1;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// y * sigmoid(y / log2 e) without the ln2 factor: y / (1 + 2^-y)
__device__ __forceinline__ float silu_log2(float y) {
  return y * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-y));
}

// OHALF: the output goes out in half precision (the step's own matrix between the attention and the second
// LayerNorm) instead of bf16 (what a caller of the attention alone gets).  TURNS: see the tile loop.
template <bool OHALF, bool TURNS>
__global__ __launch_bounds__(256, 4) void attention_bf16_mfma(HstuDims hd, uint32_t layer, const uint16_t* __restrict__ q,
                                                              const float* __restrict__ pos,
                                                              const float* __restrict__ time, KvView kv,
                                                              const uint32_t* __restrict__ ts_marks, uint32_t epoch,
                                                              const AttnItem* __restrict__ items,
                                                              const AttnWork* __restrict__ work,
                                                              AttnDies dies,
                                                              float* __restrict__ partials,
                                                              const int32_t* __restrict__ page_tables,
                                                              const long long* __restrict__ ts,
                                                              uint16_t* __restrict__ o) {
  __shared__ __attribute__((aligned(16))) AttnShared sm;
  const uint32_t tid = threadIdx.x, lane = tid & 63, g = lane >> 5, li = lane & 31;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto scalar = [](uint32_t x) { return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(x)); };  // all lanes agree on it
  const uint32_t die = blockIdx.x % kXcds, at = dies.begin[die] + blockIdx.x / kXcds;
  if (at >= dies.begin[die + 1]) return;
  const AttnWork wk = work[at];
  const AttnItem item = items[wk.item_head >> 4];
  const uint32_t h = scalar(wk.item_head & 15);
  const uint32_t P = scalar(item.prefix_len), T = scalar(item.new_len), S = P + T;
  const uint32_t q0 = item.qt * kAttnQ;  // first query (index among the new tokens) of the block
  const long long* tsr = ts + item.ts_off;
  const long long ts_base = tsr[0];
  const long long span = tsr[S - 1] - ts_base;
  // 32-bit times relative to the request's first: only for requests whose timestamps never decrease
  const bool fast = hd.n_time <= 32 && ts_marks[item.req] != epoch && span >= 0 && span < (1ll << 31);
  if (tid < 64) sm.time[tid] = tid < hd.n_time ? time[(static_cast<uint64_t>(layer) * hd.H + h) * hd.n_time + tid] : 0.0f;
  if (tid >= 64 && tid < 96) {
    const uint32_t bkt = 95 - tid;  // floor(log2(gap)) of a gap with tid - 64 leading zeros
    sm.rtime[tid - 64] = time[(static_cast<uint64_t>(layer) * hd.H + h) * hd.n_time + (bkt < hd.n_time - 1 ? bkt : hd.n_time - 1)];
  }
  // (a pointer made of integers: that it is global memory has to be said)
  typedef __attribute__((address_space(1))) const uint8_t* GlobalBytes;
  typedef __attribute__((address_space(1))) const float* GlobalFloats;
  const GlobalBytes pos_h = (GlobalBytes)in_scalar(reinterpret_cast<const uint8_t*>(pos + (static_cast<uint64_t>(layer) * hd.H + h) * hd.n_pos));

  // A wavefront takes 32 queries and all keys of a tile.  With at most 64 queries in the block, the wavefronts are
  // paired instead: each pair takes 32 queries, one of it the first and the other the second half of every tile, and their
  // sums are added at the end, so that no SIMD idles (128 requests of 64 queries: 122 -> 108 us).
  const bool paired = T - q0 <= 64;
  const uint32_t grp = paired ? wave & 1 : wave;
  const uint32_t ql = 32 * grp + li;  // query index inside the block
  const uint32_t qi = q0 + ql;
  const bool q_ok = qi < T;
  const uint32_t p = P + qi;
  const uint32_t first = q0 + 32 * grp;
  const bool grp_active = first < T;
  const uint32_t halves = scalar(!grp_active ? 0 : paired ? 1 << (wave >> 1) : 3);  // the half tiles that are the wavefront's, a bit each
  const uint32_t grp_first = P + first, grp_last = P + (first + 31 < T - 1 ? first + 31 : T - 1);
  const uint32_t tq = static_cast<uint32_t>((q_ok ? tsr[p] : ts_base) - ts_base);
  uint32_t tq_first = 0, tq_last = 0;
  if (grp_active) {
    tq_first = static_cast<uint32_t>(tsr[grp_first] - ts_base);
    tq_last = static_cast<uint32_t>(tsr[grp_last] - ts_base);
  }
  tq_first = __builtin_amdgcn_readfirstlane(tq_first);
  tq_last = __builtin_amdgcn_readfirstlane(tq_last);
  bf16x8 qf[4];  // Q^T operand: lane (g, li) holds query li, d_h elements 16*st + 8*g .. +8
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    u32x4 val = {0, 0, 0, 0};
    if (q_ok) val = *reinterpret_cast<const u32x4*>(q + static_cast<uint64_t>(item.x_off + qi) * hd.d + h * 64 + 16 * st + 8 * g);
    qf[st] = __builtin_bit_cast(bf16x8, val);
  }
  f32x16 oacc[2];
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
    for (int e = 0; e < 16; ++e) oacc[b2][e] = 0.0f;

  const uint64_t koff = kv_block_offset(hd, layer, 0, h, 2), voff = kv_block_offset(hd, layer, 1, h, 2);
  const uint8_t* const k_head = in_scalar(kv.base + koff);  // the head's keys and values in page 0
  const uint8_t* const v_head = in_scalar(kv.base + voff);
  const uint32_t kt_begin = scalar(wk.k) * dies.piece;
  const uint32_t kt_end = scalar(wk.k + 1 == item.pieces ? attn_tiles(item) : kt_begin + dies.piece);
  // the item's slice of the page table goes to LDS once, so that a tile fetch is a single
  // global round trip instead of two dependent ones
  uint32_t page0, unused_ip;
  split_token(hd, kt_begin * 64, &page0, &unused_ip);
  {
    const uint32_t last_key = (kt_end * 64 < S ? kt_end * 64 : S) - 1;
    uint32_t page_last;
    split_token(hd, last_key, &page_last, &unused_ip);
    for (uint32_t i = tid; i <= page_last - page0 && i < kAttnMaxItemPages; i += 256) {
      int32_t pg = page_tables[item.page_table_off + page0 + i];
      if (pg < 0 || static_cast<uint32_t>(pg) >= kv.n_pages) {
        atomicAdd(&kv.counters[ctr_index(kCtrBadPages)], 1ull);
        pg = -1;
      }
      sm.pages[i] = pg;
    }
    if (tid == 0) sm.pages[kAttnMaxItemPages - 1] = -1;
  }
  // Positional window: entry x = (key - first key of the item) + (127 - query in the block) holds the (reversed, scaled)
  // bias of the distance between that query and the item's first key, less x.
  const PosEntries pe = pos_entries(P + q0 + kAttnQ - 1 - kt_begin * 64, hd.n_pos);
  const GlobalBytes pos_0 = pos_h + 4 * pe.base;
  auto pos_at = [&](uint32_t x0, uint32_t x) {  // entry x0 + x
    return *(GlobalFloats)(pos_0 + min(max(pe.first - x0 - x, 256u), pe.last) * 4u);
  };
  auto pos_put_copy = [&](uint32_t s, uint32_t x, float v, bool mirror) {
    const uint32_t at = (x - s) & (kPosRing - 1);
    sm.pos[s][at] = v;
    if (mirror && at < kPosMirror) sm.pos[s][kPosRing + at] = v;
  };
  // Key times: the low half as loaded, and what the tile keeps of it.  (Apart, so that nothing waits for the load where it
  // is issued: there the wait held up the wavefront's copies of the tile by a round trip to memory.)  Keys past the end of the
  // sequence come after every query: the causal select removes them, whatever their time.
  auto time_low = [&](uint32_t j) { return reinterpret_cast<const uint32_t*>(tsr)[2 * static_cast<uint64_t>(min(j, S - 1))]; };
  auto relative_time = [&](uint32_t low) { return low - static_cast<uint32_t>(ts_base); };
  if (tid < 255) {  // of the first two tiles
    const float v = pos_at(0, tid);
#pragma unroll
    for (uint32_t s = 0; s < 4; ++s) pos_put_copy(s, tid, v, true);
  }
  if (tid >= 128) (&sm.tk[0][0])[tid - 128] = relative_time(time_low(kt_begin * 64 + tid - 128));
  __syncthreads();

  // A tile is copied global -> LDS without passing through registers, four 1 KB copies per wavefront: two of K, two of V^T.
  // A lane's 16 bytes of copy i: LDS row 16 * wave + 8 * i + r with r = lane / 8, chunk position lane % 8, chunk part ^ 4 i.
  // LDS row R of K holds key R with bits 2 and 3 swapped: the 8 keys a lane holds after the first product are then
  // consecutive, and the matching V^T operand is one 16-byte read.
  const uint32_t r8 = lane >> 3, part = (lane & 7) ^ (r8 >> 1);
  const uint32_t krow = 16 * wave + (r8 & 3) + 8 * (r8 >> 2);  // + 4 i
  const uint32_t vrow = 16 * wave + r8;                        // + 8 i
  const uint32_t kconst = krow * 128 + part * 16, vconst = (vrow * hd.pt + part * 8) * 2;
  const bool one_page_tiles = hd.pt_shift < 32 && hd.pt >= 64;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(&sm.kv[0][0][0])) + wave * 2048;
  // The page of a tile, or -1 if it may sit in several.  It is read a tile ahead, beside other LDS reads that are waited for
  // there, so that the copies of a tile start right behind the barrier.  (Asked for tiles up to the second behind the item's last one,
  // whose word exists but may hold anything: kAttnSparePages.)
  const uint32_t whole_tiles = one_page_tiles ? S / 64 : 0;  // tiles before this one sit in one page each, inside the sequence
  auto page_of = [&](uint32_t kt) -> int32_t { return sm.pages[kt < whole_tiles ? ((kt * 64) >> hd.pt_shift) - page0 : kAttnMaxItemPages - 1]; };
  auto fetch = [&](uint32_t kt, uint32_t buf, int32_t page) {
    const uint32_t j0 = kt * 64;
    const uint32_t lds = lds0 + buf * 16384;
    if (page >= 0) {  // the whole tile sits in one page and inside the sequence: scalar bases, no per-lane arithmetic
      const uint32_t tb = j0 & (hd.pt - 1);
      const uint64_t pb = static_cast<uint64_t>(page) * kv.page_size;
      const uint8_t* kbase = k_head + pb + static_cast<uint64_t>(tb) * 128;
      const uint8_t* vbase = v_head + pb + static_cast<uint64_t>(tb) * 2;
      copy_to_lds<1>(lds, kbase, kconst);
      copy_to_lds<1>(lds + 1024, kbase + 512, kconst ^ 64);
      copy_to_lds<1>(lds + 8192, vbase, vconst);
      copy_to_lds<1>(lds + 8192 + 1024, vbase + 16 * hd.pt, vconst ^ 64);
      return;
    }
    // (The block's base passes through an empty asm, so that its sum with a lane's place in the block, the same for every
    // tile, is not kept in registers over the whole loop.)
    auto block_of = [&](uint32_t j, uint64_t off, uint32_t* ip) -> const uint8_t* {
      if (j >= S) return nullptr;
      uint32_t pi;
      split_token(hd, j, &pi, ip);
      const int32_t page = sm.pages[pi - page0];
      if (page < 0) return nullptr;
      const uint8_t* b = kv.base + static_cast<uint64_t>(page) * kv.page_size + off;
      asm volatile("" : "+v"(b));
      return b;
    };
    const uint8_t* zero = reinterpret_cast<const uint8_t*>(&kZeroChunk);
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i) {
      uint32_t ip = 0;
      const uint8_t* kb = block_of(j0 + krow + 4 * i, koff, &ip);
      const uint8_t* src = kb ? kb + (ip * 128 + (part ^ 4 * i) * 16) : zero;
      copy_to_lds_from(lds + i * 1024, src);
    }
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i) {  // V^T: 8 consecutive keys inside one page (page_tokens % 8 == 0)
      uint32_t ip = 0;
      const uint8_t* vb = block_of(j0 + (part ^ 4 * i) * 8, voff, &ip);
      const uint8_t* src = vb ? vb + ((vrow + 8 * i) * hd.pt + ip) * 2 : zero;
      copy_to_lds_from(lds + 8192 + i * 1024, src);
    }
  };
  // Behind the copies: keys past the end of the sequence that share a chunk of V^T with the last ones hold whatever the
  // page held before, and are cleared by the lane that copied them.
  auto fetched = [&](uint32_t kt, uint32_t buf) {
    const uint32_t j0 = kt * 64;
    if (j0 + 64 <= S || (S & 7) == 0) return;
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i) {
      const uint32_t j = j0 + (part ^ 4 * i) * 8;
      if (j < S && j + 8 > S) {
        u32x4* c = reinterpret_cast<u32x4*>(&sm.kv[buf][1][wave * 2048 + i * 1024 + lane * 16]);
        u32x4 v = *c;
#pragma unroll
        for (uint32_t e = 0; e < 8; ++e)
          if (j + e >= S) v[e >> 1] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
        *c = v;
      }
    }
  };

  // operand reads: row li (+ 32) of a tile, chunk 2 * st + g
  uint32_t chunk_off[4];
#pragma unroll
  for (uint32_t st = 0; st < 4; ++st) chunk_off[st] = li * 128 + 16 * ((2 * st + g) ^ (li >> 1 & 7));
  const uint32_t pos_c0 = 8 * g + 127 - ql;  // the lane's first window entry of the item's first half tile
  const uint8_t* pos_copy = reinterpret_cast<const uint8_t*>(sm.pos[pos_c0 & 3]);
  const uint32_t pos_c = (pos_c0 & ~3u) * 4;

  // both buffers are free at first: two tiles are on their way at once (items of small steps have two)
  int32_t next_page = __builtin_amdgcn_readfirstlane(page_of(kt_begin + 1));
  fetch(kt_begin, 0, __builtin_amdgcn_readfirstlane(page_of(kt_begin)));
  if (kt_begin + 1 < kt_end) {
    fetch(kt_begin + 1, 1, next_page);
    wait_vm<4>();  // the first tile's: whatever the path, the second one's are four copies behind them
  } else {
    wait_vm<0>();
  }
  fetched(kt_begin, 0);
  // (the general requests have a loop of their own, so that what it needs does not weigh on the other's registers)
  auto sweep = [&](auto fast_tag) {
    constexpr bool FAST = decltype(fast_tag)::value;
    // Two tiles per turn of the loop: the buffer is a constant of the code, and addresses in LDS are the same for every tile.
    // (2: any tile, for the general requests.)
    auto tile = [&](uint32_t kt, auto half_tag) {
      constexpr uint32_t HALF = decltype(half_tag)::value;
      uint32_t t = kt - kt_begin;
      asm volatile("" : "+s"(t));  // (opaque: what follows from it is scalar, or one vector instruction, instead of a register that steps along)
      const uint32_t j0 = (kt_begin + t) * 64;
      const uint32_t buf = HALF < 2 ? HALF : t & 1;
      // one barrier per tile: tile kt is in LDS, and every wavefront is done with tile kt - 1, whose half takes tile kt + 1
      __syncthreads();
      // The four blocks of a CU take turns at going first, one tile each: left to itself a SIMD serves its older wavefronts
      // first, and of blocks that start together with equal work the last ends half as much later again as the first, with
      // nothing beside it to cover its latencies (32 x 512 queries behind 16 384 keys, d = 512: 0.88 ms, now 0.83).  Not where
      // the launch's last round is mostly empty (AttnSchedule::ends_evenly).
      if constexpr (TURNS) {
        if (t & 2) {
          if (buf) __builtin_amdgcn_s_setprio(0);
          else __builtin_amdgcn_s_setprio(1);
        } else {
          if (buf) __builtin_amdgcn_s_setprio(2);
          else __builtin_amdgcn_s_setprio(3);
        }
      }
      const bool more = kt + 1 < kt_end;
      // The next tile's 64 window entries, which every wavefront puts into one of the four copies, and its timestamps, which
      // the wavefronts bring in turn: no SIMD has more of this to do than another.
      float next_pos = 0.0f;
      uint32_t next_time = 0;
      auto bring = [&]() {
        if (!more || t == 0) return;
        next_pos = pos_at(64 * t, 191 + lane);
        if (wave == (t & 3)) next_time = time_low(j0 + 64 + lane);
        fetch(kt + 1, buf ^ 1, next_page);
      };
      const uint8_t* ks = &sm.kv[buf][0][0];
      const uint8_t* vs = &sm.kv[buf][1][0];
      const int32_t page_after = page_of(kt_begin + t + 2);
      const uint32_t key_time = FAST ? sm.tk[buf][lane] : 0;
      auto k_frag = [&](int sb, int st) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ks + sb * 4096 + chunk_off[st])); };
      auto v_frag = [&](int sb, int s2, int db) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(vs + db * 4096 + chunk_off[2 * sb + s2]));
      };
      // S^T = K Q^T on top of the positional bias: lane's window entries x0 .. x0+7 and x0+16 .. x0+23
      auto scores_begin = [&](int sb) {
        const float* pw = reinterpret_cast<const float*>(pos_copy + ((pos_c + 256 * t + 128 * sb) & (4 * kPosRing - 1)));
        const f32x4 w0 = *reinterpret_cast<const f32x4*>(pw), w1 = *reinterpret_cast<const f32x4*>(pw + 4);
        const f32x4 w2 = *reinterpret_cast<const f32x4*>(pw + 16), w3 = *reinterpret_cast<const f32x4*>(pw + 20);
        f32x16 sacc;
  #pragma unroll
        for (int e = 0; e < 4; ++e) {
          sacc[e] = w0[e];
          sacc[4 + e] = w1[e];
          sacc[8 + e] = w2[e];
          sacc[12 + e] = w3[e];
        }
        return sacc;
      };
      // bias, SiLU, mask -> bf16 pairs.  sacc[e]: key kb + 16*(e/8) + 8*g + e%8, query li;
      // y = (q.k + pos) * log2 e
      auto epilogue = [&](int sb, const f32x16& sacc, uint32_t (&pk)[8]) {
        const uint32_t kb = j0 + 32 * sb;
        const bool diag = kb + 31 > grp_first;
        int mode = 2;  // 0: one time bias for the block, 1: two adjacent buckets, 2: bucket per score (+ mask)
        float c_lo = 0.0f, c_hi = 0.0f;
        uint32_t thr = 0;
        if (FAST && !diag) {
          const uint32_t tk_first = __builtin_amdgcn_readlane(key_time, 32 * sb), tk_last = __builtin_amdgcn_readlane(key_time, 32 * sb + 31);
          const uint32_t gap_min = tq_first - tk_last, gap_max = tq_last - tk_first;
          const uint32_t bmin = bucket_u32(gap_min, hd.n_time);
          const uint32_t bmax = bucket_u32(gap_max, hd.n_time);
          c_lo = sm.time[bmin];
          if (bmin == bmax) {
            mode = 0;
          } else if (bmax == bmin + 1) {
            mode = 1;
            c_hi = sm.time[bmax];
            thr = 2u << bmin;  // gaps >= 2^(bmin+1) belong to the upper bucket
          }
        }
        if (mode == 0) {
  #pragma unroll
          for (int e = 0; e < 16; e += 2)
            pk[e >> 1] = pack_bf16x2(silu_log2(sacc[e] + c_lo), silu_log2(sacc[e + 1] + c_lo));
          return;
        }
        const int lim = static_cast<int>(p) - static_cast<int>(kb) - 8 * static_cast<int>(g);  // visible: key offset <= lim
        if (FAST) {
          // eight scores at a time: the lane's key timestamps (all below 2^31) come as two 16-byte reads
          const u32x4* tkp = reinterpret_cast<const u32x4*>(&sm.tk[buf][32 * sb + 8 * g]);
          const int32_t lim_t = tq >= thr ? static_cast<int32_t>(tq - thr) : -1;
  #pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            const u32x4 t0 = tkp[4 * hf], t1 = tkp[4 * hf + 1];
            const uint32_t tkl[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
            float a[8];
            if (mode == 1) {
              // gap >= thr  <=>  key time <= query time - thr (never, if that is negative)
  #pragma unroll
              for (int e = 0; e < 8; ++e)
                a[e] = silu_log2(sacc[8 * hf + e] + (static_cast<int32_t>(tkl[e]) <= lim_t ? c_hi : c_lo));
            } else {
              // bucket per score through the table indexed by the gap's leading zero count; a key after
              // the query gives a wrapped gap, whose (valid) table entry the causal select discards
  #pragma unroll
              for (int e = 0; e < 8; ++e) {
                const uint32_t gap = tq - tkl[e];
                a[e] = silu_log2(sacc[8 * hf + e] + sm.rtime[__clz(static_cast<int>(gap > 1 ? gap : 1))]);
              }
              if (diag) {
  #pragma unroll
                for (int e = 0; e < 8; ++e) a[e] = 16 * hf + e <= lim ? a[e] : 0.0f;
              }
            }
  #pragma unroll
            for (int e = 0; e < 8; e += 2) pk[4 * hf + (e >> 1)] = pack_bf16x2(a[e], a[e + 1]);
          }
          return;
        }
        // 64-bit gaps (requests spanning 2^31 s or more or with decreasing timestamps, or more than 32 buckets)
        const long long ts_q = q_ok ? tsr[p] : ts_base;
  #pragma unroll
        for (int e = 0; e < 16; e += 2) {
          float a[2];
  #pragma unroll
          for (int k = 0; k < 2; ++k) {
            const int off = 16 * ((e + k) / 8) + ((e + k) % 8);
            const uint32_t jl = 32 * sb + off + 8 * g;
            const uint32_t bkt = time_bucket(ts_q - (j0 + jl < S ? tsr[j0 + jl] : ts_base), hd.n_time);
            const float v = silu_log2(sacc[e + k] + sm.time[bkt]);
            a[k] = off <= lim ? v : 0.0f;
          }
          pk[e >> 1] = pack_bf16x2(a[0], a[1]);
        }
      };
      // O^T += V^T P^T; the P^T operand of step s2 = elements 8*s2 .. 8*s2+7: keys kb + 16*s2 + 8*g + 0..7
      auto accumulate = [&](int sb, const uint32_t (&pk)[8]) {
  #pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const bf16x8 pf = __builtin_bit_cast(bf16x8, u32x4{pk[4 * s2], pk[4 * s2 + 1], pk[4 * s2 + 2], pk[4 * s2 + 3]});
  #pragma unroll
          for (int db = 0; db < 2; ++db)
            oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_frag(sb, s2, db), pf, oacc[db], 0, 0, 0);
        }
      };
  #pragma unroll
      for (uint32_t sb = 0; sb < 2; ++sb) {
        // (General requests read times from memory for each score and wait for all that is on its way: the copies go out in front,
        // where the two wavefronts of a pair wait for them side by side.  128 x 64 behind 3072: between the halves 935 us, so 811.)
        if (sb == (FAST ? 1 : 0)) bring();
        if (!(halves >> sb & 1) || j0 + 32 * sb > grp_last) continue;  // the wavefront's, and some pair visible
        f32x16 s = scores_begin(sb);
  #pragma unroll
        for (int st = 0; st < 4; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(sb, st), qf[st], s, 0, 0, 0);
        uint32_t pk[8];
        epilogue(sb, s, pk);
        accumulate(sb, pk);
      }
      next_page = __builtin_amdgcn_readfirstlane(page_after);
      uint32_t at = t;  // (the conditions are computed again: carried through the tile they take vector registers)
      asm volatile("" : "+s"(at));
      if (at + 1 < kt_end - kt_begin) {
        wait_vm<0>();
        fetched(kt + 1, buf ^ 1);
        if (at == 0) return;  // (the second tile's window and times came with the first's)
        pos_put_copy(wave, 64 * at + 191 + lane, next_pos, buf == 1 && (at & 2) == 0);  // (only such tiles bring the ring's first entries)
        if (wave == (at & 3)) sm.tk[buf ^ 1][lane] = relative_time(next_time);
      }
    };
    if constexpr (FAST) {
      for (uint32_t kt = kt_begin;;) {
        tile(kt, std::integral_constant<uint32_t, 0>{});
        if (++kt == kt_end) break;
        tile(kt, std::integral_constant<uint32_t, 1>{});
        if (++kt == kt_end) break;
      }
    } else {
      for (uint32_t kt = kt_begin; kt < kt_end; ++kt) tile(kt, std::integral_constant<uint32_t, 2>{});
    }
  };
  if (fast) sweep(std::true_type{});
  else sweep(std::false_type{});
  if (paired) {  // the second half tiles' sums join the first ones'
    __syncthreads();
    float* xs = reinterpret_cast<float*>(&sm.kv[0][0][0]) + grp * (32 * 64) + lane * 4;  // [e / 4][lane][4] per group
    if (wave >= 2) {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        *reinterpret_cast<f32x4*>(xs + 256 * k) = f32x4{oacc[k >> 2][4 * (k & 3)], oacc[k >> 2][4 * (k & 3) + 1], oacc[k >> 2][4 * (k & 3) + 2], oacc[k >> 2][4 * (k & 3) + 3]};
    }
    __syncthreads();
    if (wave >= 2) return;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(xs + 256 * k);
#pragma unroll
      for (int e = 0; e < 4; ++e) oacc[k >> 2][4 * (k & 3) + e] += v[e];
    }
  }
  // oacc[db][e]: d_h element 32*db + 8*(e/4) + 4*g + e%4 of the lane's query; undo the log2 e scaling, apply 1/n
  const float sc = hd.inv_n * kLn2;
  if (item.pieces > 1) {
    // a piece of a query tile: fp32 partial [slot][query][d_h], summed by attention_reduce
    if (!q_ok) return;
    float* prow = partials + (static_cast<uint64_t>(item.slot0 + h * item.pieces + wk.k) * kAttnQ + ql) * 64;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        *reinterpret_cast<f32x4*>(prow + 32 * db + 8 * e4 + 4 * g) =
            f32x4{oacc[db][4 * e4] * sc, oacc[db][4 * e4 + 1] * sc, oacc[db][4 * e4 + 2] * sc, oacc[db][4 * e4 + 3] * sc};
  } else if (q_ok) {
    uint16_t* orow = o + static_cast<uint64_t>(item.x_off + qi) * hd.d + h * 64;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        uint2 w;
        if (OHALF) {
          w.x = pack2_f16(oacc[db][4 * e4] * sc, oacc[db][4 * e4 + 1] * sc);
          w.y = pack2_f16(oacc[db][4 * e4 + 2] * sc, oacc[db][4 * e4 + 3] * sc);
        } else {
          w.x = pack_bf16x2(oacc[db][4 * e4] * sc, oacc[db][4 * e4 + 1] * sc);
          w.y = pack_bf16x2(oacc[db][4 * e4 + 2] * sc, oacc[db][4 * e4 + 3] * sc);
        }
        *reinterpret_cast<uint2*>(orow + 32 * db + 8 * e4 + 4 * g) = w;
      }
  }
}

// Sum the fp32 partials of a query tile that was cut, in the order of their slots, and write the output.
__global__ __launch_bounds__(256) void attention_reduce(HstuDims hd, const AttnItem* __restrict__ items,
                                                        const uint32_t* __restrict__ groups,
                                                        const float* __restrict__ partials, uint16_t* __restrict__ o,
                                                        uint32_t o_half) {
  // blockIdx.x = cut query tile and head; blockIdx.y = which 16 of the tile's query rows: a thread owns one 16-byte piece of
  // one row, so that the pieces' loads of a whole tile are in flight at once
  const AttnItem it = items[groups[blockIdx.x / hd.H]];
  const uint32_t h = blockIdx.x % hd.H;
  const uint32_t row = blockIdx.y * 16 + threadIdx.x / 16, c4 = threadIdx.x & 15;
  const uint32_t qi = it.qt * kAttnQ + row;
  if (qi >= it.new_len) return;
  const float* src = partials + (static_cast<uint64_t>(it.slot0 + h * it.pieces) * kAttnQ + row) * 64 + 4 * c4;
  constexpr uint64_t step = kAttnQ * 64;  // from one piece's partial to the next
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  auto add = [&](const float4& v) { acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w; };
  uint32_t k = 0;
  for (; k + 4 <= it.pieces; k += 4) {  // four loads in flight (eight: 126 tiles of a few partials 7.2 us, so 6.0)
    float4 v[4];
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const float4*>(src + (k + e) * step);
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) add(v[e]);
  }
  const uint32_t rest = it.pieces - k;  // up to three, asked for together as well (13 ragged prefills 96.3 -> 95.1 us)
  float4 v[3];
#pragma unroll
  for (uint32_t e = 0; e < 3; ++e)
    if (e < rest) v[e] = *reinterpret_cast<const float4*>(src + (k + e) * step);
#pragma unroll
  for (uint32_t e = 0; e < 3; ++e)
    if (e < rest) add(v[e]);
  uint2 w;
  if (o_half) {
    w.x = pack2_f16(acc.x, acc.y);
    w.y = pack2_f16(acc.z, acc.w);
  } else {
    w.x = pack2_bf16(acc.x, acc.y);
    w.y = pack2_bf16(acc.z, acc.w);
  }
  *reinterpret_cast<uint2*>(o + static_cast<uint64_t>(it.x_off + qi) * hd.d + h * 64 + 4 * c4) = w;
}

// The same sums, in the same order, for few tiles of many partials (sums_by_rows): a wavefront sums one row, a lane one float of
// it, and asks for 32 partials at a time, 16 where no more are left (a round that has fewer asks for the last one again).  They
// come from other dies' launches, through memory, and what counts there is how often that is waited for.
__global__ __launch_bounds__(256) void attention_reduce_rows(HstuDims hd, const AttnItem* __restrict__ items,
                                                             const uint32_t* __restrict__ groups,
                                                             const float* __restrict__ partials, uint16_t* __restrict__ o,
                                                             uint32_t o_half) {
  const AttnItem it = items[groups[blockIdx.x / hd.H]];
  const uint32_t h = blockIdx.x % hd.H, col = threadIdx.x & 63;
  const uint32_t row = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t qi = it.qt * kAttnQ + row;
  if (qi >= it.new_len) return;  // the whole wavefront
  const float* src = partials + (static_cast<uint64_t>(it.slot0 + h * it.pieces) * kAttnQ + row) * 64 + col;
  constexpr uint64_t step = kAttnQ * 64;
  float acc = 0.0f;
  uint32_t k = 0;
  auto round = [&](auto n) {
    constexpr uint32_t kN = decltype(n)::value;
    float v[kN];
#pragma unroll
    for (uint32_t e = 0; e < kN; ++e) v[e] = src[min(k + e, it.pieces - 1) * step];
#pragma unroll
    for (uint32_t e = 0; e < kN; ++e) acc = k + e < it.pieces ? acc + v[e] : acc;
    k += kN;
  };
  while (k < it.pieces) {
    if (it.pieces - k > 16) round(std::integral_constant<uint32_t, 32>{});
    else round(std::integral_constant<uint32_t, 16>{});
  }
  const float right = __shfl_xor(acc, 1);
  if ((col & 1) == 0)
    *reinterpret_cast<uint32_t*>(o + static_cast<uint64_t>(it.x_off + qi) * hd.d + h * 64 + col) = o_half ? pack2_f16(acc, right) : pack2_bf16(acc, right);
}

// Are a request's timestamps non-decreasing?  A block looks at tokens 2048 c + 1 .. 2048 (c + 1) of requests r0, r0 + stride, ..
// (eight per thread, all loads independent).  The first block that finds a decrease marks and counts the request.
constexpr uint32_t kTsChunk = 2048;
template <typename GetReq>
__device__ __forceinline__ void check_timestamps(const GetReq& req, uint32_t B, uint32_t c, uint32_t r0, uint32_t stride,
                                                 uint32_t* __restrict__ marks, uint32_t epoch, const long long* __restrict__ ts,
                                                 unsigned long long* __restrict__ counters) {
  for (uint32_t r = r0; r < B; r += stride) {  // (the grid's second dimension stops at 65 535)
    const ReqDev rq = req(r);
    const uint32_t S = rq.prefix_len + rq.new_len;
    const uint32_t j0 = c * kTsChunk + 1;
    if (j0 >= S) continue;  // uniform over the block
    const long long* t = ts + rq.ts_off;
    bool bad = false;
#pragma unroll
    for (uint32_t k = 0; k < kTsChunk / 256; ++k) {
      const uint32_t j = j0 + k * 256 + threadIdx.x;
      if (j < S) bad |= t[j] < t[j - 1];
    }
    if (__syncthreads_or(bad) && threadIdx.x == 0) {
      if (atomicExch(&marks[r], epoch) != epoch) atomicAdd(&counters[ctr_index(kCtrUnorderedTs)], 1ull);
    }
  }
}
// The lists (the requests first) lie in pinned host memory: the grid copies them to the device, 16 KB per block and pass
// with every load in flight, while it checks the timestamps.  A copy command in front of the kernel took 13 us of the
// stream (64 KB and more; 3.5 for less); the kernel takes the 7 us (128 x 3136 tokens) that it took without the copy: both are
// bound by one round trip.  (Loads at system scope, one by one, would make it 147 us.  Plain ones see what the host wrote
// before the launch, and the host waits for the kernel before it writes the buffer again.)
constexpr uint32_t kCopyAhead = 4;
__global__ __launch_bounds__(256) void begin_step(const uint4* __restrict__ src, uint4* __restrict__ dst, uint32_t n16, uint32_t B,
                                                  uint32_t* __restrict__ marks, uint32_t epoch, const long long* __restrict__ ts,
                                                  unsigned long long* __restrict__ counters) {
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * gridDim.y * 256;
  const uint64_t first = (static_cast<uint64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
  for (uint64_t i0 = first; i0 < n16; i0 += kCopyAhead * stride) {
    uint4 v[kCopyAhead];
#pragma unroll
    for (uint32_t k = 0; k < kCopyAhead; ++k) {
      const uint64_t i = i0 + k * stride;
      v[k] = i < n16 ? src[i] : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (uint32_t k = 0; k < kCopyAhead; ++k) {
      const uint64_t i = i0 + k * stride;
      if (i < n16) dst[i] = v[k];
    }
  }
  if (ts) check_timestamps([&](uint32_t r) { return reinterpret_cast<const ReqDev*>(src)[r]; }, B, blockIdx.x, blockIdx.y, gridDim.y, marks, epoch, ts, counters);
}
// The same for a small step, whose lists (the requests first) come as an argument: no copy engine, no staging buffer to
// wait for (10 us of host time and 5 us of the stream's a step).
__global__ __launch_bounds__(256) void begin_step_with_lists(ListArg arg, uint4* __restrict__ dst, uint32_t n16, uint32_t B,
                                                             uint32_t* __restrict__ marks, uint32_t epoch,
                                                             const long long* __restrict__ ts, unsigned long long* __restrict__ counters) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < n16) dst[threadIdx.x] = reinterpret_cast<const uint4*>(arg.bytes)[threadIdx.x];
  if (ts) check_timestamps([&](uint32_t r) { return reinterpret_cast<const ReqDev*>(arg.bytes)[r]; }, B, blockIdx.x, blockIdx.y, gridDim.y, marks, epoch, ts, counters);
}
// The same again beside the first layer's front half, for joined halves: blocks from first_block on begin the step, the others,
// which read the requests out of the argument, are layer_join's.  One kernel less in the chain of a small step: one request of
// 64 behind 2973, pass 101 -> 98 us, 13 ragged prefills 108 -> 105.5.
struct BeginArgs {
  uint32_t first_block, chunks, B, n16, group_req_at;
  uint32_t epoch;
  uint32_t* marks;
  uint4* dst;
  const long long* ts;
  unsigned long long* counters;
};
template <int KD>
__global__ __launch_bounds__(256, KD <= 256 ? 2 : 1) void layer_first(JoinArgs a, BeginArgs b, ListArg arg) {
  const ReqDev* reqs = reinterpret_cast<const ReqDev*>(arg.bytes);
  if (blockIdx.x >= b.first_block) {
    const uint32_t i = blockIdx.x - b.first_block;
    if (i == 0 && threadIdx.x < b.n16) b.dst[threadIdx.x] = reinterpret_cast<const uint4*>(arg.bytes)[threadIdx.x];
    check_timestamps([&](uint32_t r) { return reqs[r]; }, b.B, i % b.chunks, i / b.chunks, b.B, b.marks, b.epoch, b.ts, b.counters);
    return;
  }
  layer_join_block<KD, false, true>(a, reqs, reinterpret_cast<const uint32_t*>(arg.bytes + b.group_req_at));
}
static_assert(kListArgBytes / 16 <= 256, "one 16-byte word of the lists per thread");

__global__ void scale_f32(const float* __restrict__ in, float* __restrict__ out, uint64_t n, float s) {
  for (uint64_t k = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; k < n;
       k += static_cast<uint64_t>(gridDim.x) * blockDim.x)
    out[k] = in[k] * s;
}

// q * log2(e) for callers that hand the attention kernel an unscaled query matrix
__global__ void scale_bf16(const uint16_t* __restrict__ in, uint16_t* __restrict__ out, uint64_t n, float s) {
  for (uint64_t k = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; k < n;
       k += static_cast<uint64_t>(gridDim.x) * blockDim.x)
    out[k] = f2bf(bf2f(in[k]) * s);
}

// Copy of a bf16 weight matrix [rows][cols] in half precision, in the order in which the fused layer halves use it as
// an MFMA operand: for every 32 columns and 16 rows one piece of 64 lanes x 8 elements, lane (g, i) holding column i
// and rows 8 g .. 8 g + 7 (exact unless a weight is below 2^-14 in magnitude).
__global__ __launch_bounds__(256) void weight_fragments(const uint16_t* __restrict__ w, uint16_t* __restrict__ wf, uint32_t rows, uint32_t cols) {
  const uint64_t n = static_cast<uint64_t>(rows) * cols / 8;  // one thread: the 8 elements of one lane
  for (uint64_t t = blockIdx.x * 256ull + threadIdx.x; t < n; t += gridDim.x * 256ull) {
    const uint32_t lane = t & 63, g = lane >> 5, li = lane & 31;
    const uint64_t piece = t >> 6;
    const uint32_t st = piece % (rows / 16), cb = piece / (rows / 16);
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = f2h(bf2f(w[static_cast<uint64_t>(16 * st + 8 * g + e) * cols + 32 * cb + li]));
    *reinterpret_cast<uint4*>(wf + 8 * t) = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
  }
}

// transposed copy of a bf16 weight matrix in half precision (exact unless a weight is below 2^-14 in magnitude)
__global__ void transpose_bf16_to_f16(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt, uint32_t rows, uint32_t cols) {
  __shared__ uint16_t tile[32][33];
  const uint32_t bx = blockIdx.x * 32, by = blockIdx.y * 32;
  for (uint32_t yy = threadIdx.y; yy < 32; yy += 8)
    if (by + yy < rows && bx + threadIdx.x < cols) tile[yy][threadIdx.x] = f2h(bf2f(w[static_cast<uint64_t>(by + yy) * cols + bx + threadIdx.x]));
  __syncthreads();
  for (uint32_t yy = threadIdx.y; yy < 32; yy += 8)
    if (bx + yy < cols && by + threadIdx.x < rows) wt[static_cast<uint64_t>(bx + yy) * rows + by + threadIdx.x] = tile[threadIdx.x][yy];
}

}  // namespace

template <typename TX, typename TY>
static void layernorm_dispatch(const HstuDims& hd, const void* x, const float* g, const float* b, const void* gate,
                               void* y, uint32_t N, hipStream_t stream) {
  const TX* xs = static_cast<const TX*>(x);
  const TY* gs = static_cast<const TY*>(gate);
  TY* ys = static_cast<TY*>(y);
  const uint32_t chunks = hd.d / 8;
  const dim3 block(256);
#define RACER_LN(LPR, KC)                                                                                        \
  hipLaunchKernelGGL((layernorm_rows<TX, TY, LPR, KC>), dim3((N + 256 / LPR - 1) / (256 / LPR)), block, 0, stream, \
                     xs, g, b, gs, ys, N, hd.d, hd.eps)
  if (chunks <= 8) RACER_LN(8, 1);
  else if (chunks <= 16) RACER_LN(16, 1);
  else if (chunks <= 32) RACER_LN(32, 1);
  else if (chunks <= 64) RACER_LN(64, 1);
  else RACER_LN(64, 2);
#undef RACER_LN
}

// bf16 models: the first LayerNorm of a layer reads the bf16 residual stream, the second one the half-precision
// attention output and gate; both write half precision (the next product's operand)
hipError_t launch_layernorm(const HstuDims& hd, const void* x, const float* g, const float* b, const void* gate,
                            void* y, uint32_t N, hipStream_t stream) {
  if (N == 0) return hipSuccess;
  if (gate) layernorm_dispatch<half_t, half_t>(hd, x, g, b, gate, y, N, stream);
  else layernorm_dispatch<bf16_t, half_t>(hd, x, g, b, gate, y, N, stream);
  return hipGetLastError();
}

bool layer_halves_fused(const HstuDims& hd) { return hd.elem == 1 && (hd.d == 64 || hd.d == 128 || hd.d == 256 || hd.d == 512); }

// How many column tiles a block of a layer half sweeps: all of them (kMaxSweep at most) as long as the row tiles fill the
// chip's block slots (the rows are then read and normalised once), and fewer for the row tiles that are left over for a
// last, partial round, so that this round is short and reaches every CU: the sweep is halved until there are 512 blocks,
// down to one tile.  (Row tiles that fill no round are all left over.)
template <bool FRONT>
static hipError_t launch_layer_half(LayerHalfArgs& a, uint32_t col_tiles, hipStream_t stream) {
  constexpr uint32_t kRows = 128;  // per block
  const uint32_t row_tiles = (a.n_rows + kRows - 1) / kRows;
  const uint32_t slots = 256 * (a.hd.d <= 256 ? 4 : 2);
  uint32_t splits = col_tiles > kMaxSweep / 32 ? 2 : 1;
  a.cb0 = col_tiles / splits;
  a.rows1 = row_tiles % (slots / splits);
  a.rows0 = row_tiles - a.rows1;
  a.blocks0 = a.rows0 * splits;
  while (splits < col_tiles && a.rows1 * splits < 512) splits *= 2;
  a.cb1 = col_tiles / splits;
  a.rows1_inv = a.rows1 ? (0x80000000u + a.rows1 - 1) / a.rows1 : 0;  // (exact quotients: rows1 < 1024, splits <= 64)
  const dim3 grid(a.blocks0 + a.rows1 * splits), block(256);
  switch (a.hd.d) {
    case 64: hipLaunchKernelGGL((layer_half_fused<64, FRONT, 4>), grid, block, 0, stream, a); break;
    case 128: hipLaunchKernelGGL((layer_half_fused<128, FRONT, 4>), grid, block, 0, stream, a); break;
    case 256: hipLaunchKernelGGL((layer_half_fused<256, FRONT, 4>), grid, block, 0, stream, a); break;
    case 512: hipLaunchKernelGGL((layer_half_fused<512, FRONT, 4>), grid, block, 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_layer_front_fused(const HstuDims& hd, uint32_t layer, const void* x, const float* ln_g,
                                    const float* ln_b, const void* w1f, const float* b1, void* u, void* q,
                                    const KvView& kv, const StepLists& sl, const int32_t* page_tables,
                                    hipStream_t stream) {
  if (sl.N == 0) return hipSuccess;
  if (!layer_halves_fused(hd)) return hipErrorInvalidValue;
  LayerHalfArgs a{};
  a.hd = hd;
  a.layer = layer;
  a.n_rows = sl.N;
  a.a_in = static_cast<const uint16_t*>(x);
  a.ln_g = ln_g;
  a.ln_b = ln_b;
  a.wf = static_cast<const uint16_t*>(w1f);
  a.bias = b1;
  a.u = static_cast<uint16_t*>(u);
  a.q = static_cast<uint16_t*>(q);
  a.kv = kv;
  a.reqs = sl.reqs;
  a.group_req = sl.group_req;
  a.page_tables = page_tables;
  return launch_layer_half<true>(a, 4 * hd.d / 32, stream);
}

hipError_t launch_layer_back_fused(const HstuDims& hd, const void* o, const void* u, const float* ln_g,
                                   const float* ln_b, const void* w2f, const float* b2, const void* x, void* y,
                                   const StepLists& sl, hipStream_t stream) {
  if (sl.N == 0) return hipSuccess;
  if (!layer_halves_fused(hd)) return hipErrorInvalidValue;
  LayerHalfArgs a{};
  a.hd = hd;
  a.n_rows = sl.N;
  a.a_in = static_cast<const uint16_t*>(o);
  a.gate = static_cast<const uint16_t*>(u);
  a.ln_g = ln_g;
  a.ln_b = ln_b;
  a.wf = static_cast<const uint16_t*>(w2f);
  a.bias = b2;
  a.resid = static_cast<const uint16_t*>(x);
  a.y = static_cast<uint16_t*>(y);
  return launch_layer_half<false>(a, hd.d / 32, stream);
}

bool layers_joined(const HstuDims& hd, uint32_t N, uint32_t B, uint64_t cached) { return layer_halves_fused(hd) && N <= join_max_rows(hd.d, N, B, cached); }

template <bool BACK, bool FRONT>
static void run_join(const JoinArgs& a, uint32_t blocks, hipStream_t stream) {
  switch (a.hd.d) {
    case 64: hipLaunchKernelGGL((layer_join<64, BACK, FRONT>), dim3(blocks), dim3(256), 0, stream, a); break;
    case 128: hipLaunchKernelGGL((layer_join<128, BACK, FRONT>), dim3(blocks), dim3(256), 0, stream, a); break;
    case 256: hipLaunchKernelGGL((layer_join<256, BACK, FRONT>), dim3(blocks), dim3(256), 0, stream, a); break;
    case 512: hipLaunchKernelGGL((layer_join<512, BACK, FRONT>), dim3(blocks), dim3(256), 0, stream, a); break;
  }
}

static uint32_t ts_chunks(uint32_t max_seq) { return max_seq < 2 ? 1 : (max_seq - 1 + kTsChunk - 1) / kTsChunk; }

bool begin_joins(const StepLists& sl, uint32_t max_seq) { return static_cast<uint64_t>(ts_chunks(max_seq)) * sl.B <= 512; }

hipError_t launch_layer_join(const HstuDims& hd, const LayerBack* back, const LayerFront* front, const void* x, const KvView& kv,
                             const StepLists& sl, const int32_t* page_tables, hipStream_t stream, const BeginStep* begin) {
  if (sl.N == 0) return hipSuccess;
  if (!layer_halves_fused(hd) || (!back && !front)) return hipErrorInvalidValue;
  JoinArgs a{};
  a.hd = hd;
  a.n_rows = sl.N;
  a.groups = (sl.N + 31) / 32;
  a.x = static_cast<const uint16_t*>(x);
  if (back) {
    a.o = static_cast<const uint16_t*>(back->o);
    a.gate = static_cast<const uint16_t*>(back->u);
    a.ln2_g = back->ln_g;
    a.ln2_b = back->ln_b;
    a.w2f = static_cast<const uint16_t*>(back->w2f);
    a.b2 = back->b2;
    a.y = static_cast<uint16_t*>(back->y);
  }
  uint32_t slices = 1;
  if (front) {
    a.layer = front->layer;
    a.ln1_g = front->ln_g;
    a.ln1_b = front->ln_b;
    a.w1f = static_cast<const uint16_t*>(front->w1f);
    a.b1 = front->b1;
    a.u = static_cast<uint16_t*>(front->u);
    a.q = static_cast<uint16_t*>(front->q);
    a.kv = kv;
    a.reqs = sl.reqs;
    a.group_req = sl.group_req;
    a.page_tables = page_tables;
    slices = join_slices(hd.d, a.groups);
    a.front_tiles = hd.d / 32 / slices;  // of four wavefronts
  }
  const uint32_t blocks = a.groups * slices;
  if (begin) {
    if (back || !front) return hipErrorInvalidValue;
    BeginArgs b{blocks, ts_chunks(begin->max_seq), sl.B, static_cast<uint32_t>((begin->list_bytes + 15) / 16),
                static_cast<uint32_t>(reinterpret_cast<const uint8_t*>(sl.group_req) - begin->list_dst), sl.epoch,
                const_cast<uint32_t*>(sl.ts_marks), reinterpret_cast<uint4*>(begin->list_dst),
                reinterpret_cast<const long long*>(begin->ts), begin->counters};
    const dim3 grid(blocks + b.chunks * sl.B);
    switch (hd.d) {
      case 64: hipLaunchKernelGGL(layer_first<64>, grid, dim3(256), 0, stream, a, b, *begin->arg); break;
      case 128: hipLaunchKernelGGL(layer_first<128>, grid, dim3(256), 0, stream, a, b, *begin->arg); break;
      case 256: hipLaunchKernelGGL(layer_first<256>, grid, dim3(256), 0, stream, a, b, *begin->arg); break;
      case 512: hipLaunchKernelGGL(layer_first<512>, grid, dim3(256), 0, stream, a, b, *begin->arg); break;
    }
    return hipGetLastError();
  }
  if (back && front) run_join<true, true>(a, blocks, stream);
  else if (back) run_join<true, false>(a, blocks, stream);
  else run_join<false, true>(a, blocks, stream);
  return hipGetLastError();
}

hipError_t launch_gemm_front(const HstuDims& hd, uint32_t layer, const void* xn, const void* w1, const float* b1,
                             void* u, void* q, const KvView& kv, const StepLists& sl, const int32_t* page_tables,
                             hipStream_t stream) {
  if (sl.N == 0) return hipSuccess;
  hipLaunchKernelGGL(gemm_front_bf16, dim3(sl.n_row_tiles, 4 * hd.d / 64), dim3(256), 0, stream, hd, layer,
                     static_cast<const uint16_t*>(xn), static_cast<const uint16_t*>(w1), b1, static_cast<uint16_t*>(u),
                     static_cast<uint16_t*>(q), kv, sl.reqs, sl.row_tiles, page_tables);
  return hipGetLastError();
}

hipError_t launch_gemm_back(const HstuDims& hd, const void* g, const void* w2, const float* b2, const void* x,
                            void* y, uint32_t N, hipStream_t stream) {
  if (N == 0) return hipSuccess;
  hipLaunchKernelGGL(gemm_back_bf16, dim3((N + 127) / 128, hd.d / 64), dim3(256), 0, stream, static_cast<const uint16_t*>(g),
                     static_cast<const uint16_t*>(w2), N, hd.d, b2, static_cast<const uint16_t*>(x), static_cast<uint16_t*>(y));
  return hipGetLastError();
}

hipError_t launch_attention(const HstuDims& hd, uint32_t layer, const void* q, const float* pos, const float* time,
                            const KvView& kv, const StepLists& sl, const int32_t* page_tables, const int64_t* ts,
                            void* o, bool o_half, hipStream_t stream) {
  if (sl.N == 0) return hipSuccess;
  const long long* t = reinterpret_cast<const long long*>(ts);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(sl.n_blocks), dim3(256), 0, stream, hd, layer, static_cast<const uint16_t*>(q), pos, time, kv,
                       sl.ts_marks, sl.epoch, sl.items, sl.work, sl.dies, sl.partials, page_tables, t, static_cast<uint16_t*>(o));
  };
  if (o_half) sl.turns ? run(attention_bf16_mfma<true, true>) : run(attention_bf16_mfma<true, false>);
  else sl.turns ? run(attention_bf16_mfma<false, true>) : run(attention_bf16_mfma<false, false>);
  return hipGetLastError();
}

hipError_t launch_attention_reduce(const HstuDims& hd, const StepLists& sl, void* o, bool o_half, hipStream_t stream) {
  if (sl.n_groups == 0) return hipSuccess;
  const uint32_t tiles = sl.n_groups * hd.H;
  auto run = [&](auto kernel, uint32_t rows) {
    hipLaunchKernelGGL(kernel, dim3(tiles, kAttnQ / rows), dim3(256), 0, stream, hd, sl.items, sl.groups, sl.partials, static_cast<uint16_t*>(o), o_half ? 1u : 0u);
  };
  if (sl.sum_rows) run(attention_reduce_rows, 4);
  else run(attention_reduce, 16);
  return hipGetLastError();
}

hipError_t launch_begin_step(const StepLists& sl, uint32_t max_seq, const int64_t* ts, unsigned long long* counters, const ListArg* arg,
                             const uint8_t* pinned, uint8_t* list_dst, uint64_t list_bytes, hipStream_t stream) {
  const uint32_t chunks = ts_chunks(max_seq);
  // blocks for the copy too, where the requests do not ask for as many
  const uint64_t copy_rows = arg ? 0 : std::min<uint64_t>(1024, (list_bytes / (256 * 16 * kCopyAhead) + chunks - 1) / chunks);
  const dim3 grid(chunks, static_cast<uint32_t>(std::max<uint64_t>(copy_rows, std::min<uint32_t>(sl.B, 65535)))), block(256);
  const long long* t = reinterpret_cast<const long long*>(ts);
  uint32_t* marks = const_cast<uint32_t*>(sl.ts_marks);
  if (arg)
    hipLaunchKernelGGL(begin_step_with_lists, grid, block, 0, stream, *arg, reinterpret_cast<uint4*>(list_dst),
                       static_cast<uint32_t>((list_bytes + 15) / 16), sl.B, marks, sl.epoch, t, counters);
  else
    hipLaunchKernelGGL(begin_step, grid, block, 0, stream, reinterpret_cast<const uint4*>(pinned),
                       reinterpret_cast<uint4*>(list_dst), static_cast<uint32_t>(list_bytes / 16), sl.B, marks, sl.epoch, t, counters);
  return hipGetLastError();
}

hipError_t launch_scale_bias(const float* in, float* out, uint64_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const uint32_t blocks = static_cast<uint32_t>((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
  hipLaunchKernelGGL(scale_f32, dim3(blocks), dim3(256), 0, stream, in, out, n, kLog2e);
  return hipGetLastError();
}

hipError_t launch_scale_q(const void* in, void* out, uint64_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const uint32_t blocks = static_cast<uint32_t>((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
  hipLaunchKernelGGL(scale_bf16, dim3(blocks), dim3(256), 0, stream, static_cast<const uint16_t*>(in),
                     static_cast<uint16_t*>(out), n, kLog2e);
  return hipGetLastError();
}

hipError_t launch_weight_copy(const void* w, void* wt, uint32_t rows, uint32_t cols, bool fragments, hipStream_t stream) {
  const uint16_t* src = static_cast<const uint16_t*>(w);
  uint16_t* dst = static_cast<uint16_t*>(wt);
  if (fragments)
    hipLaunchKernelGGL(weight_fragments, dim3((rows * cols / 8 + 255) / 256), dim3(256), 0, stream, src, dst, rows, cols);
  else
    hipLaunchKernelGGL(transpose_bf16_to_f16, dim3((cols + 31) / 32, (rows + 31) / 32), dim3(32, 8), 0, stream, src, dst, rows, cols);
  return hipGetLastError();
}

}  // namespace racer
