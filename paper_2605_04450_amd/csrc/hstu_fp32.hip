// HSTU layer kernels of fp32 models (the small configurations): LayerNorm and projection of a layer half in one kernel,
// and paged attention on tiles of 16 queries.  fp32 multiply-adds throughout.  These models run a few hundred tokens at
// a time: what bounds them is how many dependent memory round trips a step takes and how much of the chip shares the work.
// Layouts (pages, activations) are those of hstu_kernels.hip with 4-byte elements.
#include "hstu_common.h"

namespace racer {
namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---------------------------------------------------------------------------------------
// Layer halves.  FRONT: [U|V|Q|K] = SiLU(LN1(X) W1 + b1), K and V into the pages;  BACK: Y = X + (LN2(O) * U) W2 + b2.
// A block computes 64 output columns of 8 rows: a wavefront normalises its two rows into LDS (which no other wavefront
// reads: no barrier) and then owns the 64 columns of them, one per lane; the first 16 rows of W, and
// what the stores need, are already on their way during the LayerNorm.  8 rows a block give 512 blocks for 1024 tokens of a d = 64 model.
// What bounds it is a chain of memory round trips: all loads whose address is known go out first, and the requests are searched by
// ballot (four dependent loads per row, behind one another and in front of the rows, before).
// 1024 tokens, d = 64: front 7.6 us (8.2 with that search, 9 before; LayerNorm and product as two kernels, one thread per output: 4
// + 13), back 4.4 us (4.9; 4 + 9).  W 32 or 64 rows ahead instead of 16: 1 and 3% slower steps.
// ---------------------------------------------------------------------------------------
constexpr uint32_t kRowsPerWave = 2, kRowsPerBlock = 4 * kRowsPerWave, kMaxWidth = 1024, kAhead = 16;

struct HalfArgsF32 {
  HstuDims hd;
  uint32_t layer, N, B, n_out;
  const float* in;     // FRONT: X   BACK: O
  const float* gate;   // BACK: U
  const float* ln_g;
  const float* ln_b;
  const float* w;      // [d][n_out]
  const float* bias;
  float* u;            // FRONT outputs
  float* q;
  KvView kv;
  const ReqDev* reqs;
  const int32_t* page_tables;
  const float* resid;  // BACK: X
  float* y;            // BACK output
};

template <bool FRONT>
__global__ __launch_bounds__(256) void layer_half_f32(HalfArgsF32 a) {
  __shared__ __attribute__((aligned(16))) float xs[kRowsPerBlock][kMaxWidth + 4];
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t row0 = blockIdx.x * kRowsPerBlock + wave * kRowsPerWave;
  if (row0 >= a.N) return;  // (no barrier below)
  const uint32_t d = a.hd.d, col = blockIdx.y * 64 + lane;
  const bool col_ok = col < a.n_out;
  uint32_t row[kRowsPerWave];
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) row[r] = row0 + r < a.N ? row0 + r : row0;
  // What the kernel needs goes out at once, in the order in which it is needed: the first 64 columns of the rows (all there
  // are, or the first of several rounds), scale, shift and gate, W, bias and residual.
  ReqDev mine{};
  if (FRONT && a.B <= 64) mine = a.reqs[min(lane, a.B - 1)];
  const uint32_t c0 = lane < d ? lane : 0;
  float in0[kRowsPerWave], gate0[kRowsPerWave], resid[kRowsPerWave];
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) in0[r] = a.in[static_cast<uint64_t>(row[r]) * d + c0];
  const float gg0 = a.ln_g[c0], bb0 = a.ln_b[c0];
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) gate0[r] = FRONT ? 0.0f : a.gate[static_cast<uint64_t>(row[r]) * d + c0];
  const float* wc = a.w + (col_ok ? col : 0);
  float wr[kAhead];  // d is a multiple of 16
#pragma unroll
  for (uint32_t k = 0; k < kAhead; ++k) wr[k] = wc[static_cast<uint64_t>(k) * a.n_out];
  const float bias = a.bias[col_ok ? col : 0];
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) resid[r] = FRONT ? 0.0f : a.resid[static_cast<uint64_t>(row[r]) * d + (col_ok ? col : 0)];
  // Where K and V of the rows go: up to 64 requests are a lane each, the row's request one ballot away; more are searched, by
  // wavefronts with columns of K or V (1000 requests of 16, d = 128: 227 us with a search in every wavefront, so 212).  (The
  // page's number comes as a vector load, which is waited for where it is used; a scalar one every LDS read would wait for.)
  const uint32_t which = col / d, c_out = col % d;  // FRONT: 0: U, 1: V, 2: Q, 3: K
  int32_t page[kRowsPerWave];
  uint32_t tok[kRowsPerWave];
  if (FRONT && (a.B <= 64 || __any(which & 1))) {
#pragma unroll
    for (uint32_t r = 0; r < kRowsPerWave; ++r) {
      uint32_t first, table;  // of the row's request: the token that its row 0 would be, and its page table
      if (a.B <= 64) {
        const uint32_t req = __popcll(__ballot(lane < a.B && mine.x_off <= row[r])) - 1;
        first = __builtin_amdgcn_readlane(mine.prefix_len - mine.x_off, req);
        table = __builtin_amdgcn_readlane(mine.page_table_off, req);
      } else {
        const ReqDev rq = a.reqs[request_of(a.reqs, row[r], 0, a.B - 1)];
        first = rq.prefix_len - rq.x_off;
        table = rq.page_table_off;
      }
      uint32_t pi, any = 0;
      asm volatile("" : "+v"(any));
      split_token(a.hd, first + row[r], &pi, &tok[r]);
      page[r] = a.page_tables[table + pi + any];
    }
  }
  float s[kRowsPerWave], qq[kRowsPerWave];
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) s[r] = qq[r] = 0.0f;
  for (uint32_t c = lane; c < d; c += 64) {
#pragma unroll
    for (uint32_t r = 0; r < kRowsPerWave; ++r) {
      const float v = c == lane ? in0[r] : a.in[static_cast<uint64_t>(row[r]) * d + c];
      xs[wave * kRowsPerWave + r][c] = v;
      s[r] += v;
    }
  }
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) s[r] = wave_sum(s[r]) / d;  // mean
  for (uint32_t c = lane; c < d; c += 64) {
#pragma unroll
    for (uint32_t r = 0; r < kRowsPerWave; ++r) {
      const float dv = xs[wave * kRowsPerWave + r][c] - s[r];
      qq[r] += dv * dv;
    }
  }
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) qq[r] = 1.0f / sqrtf(wave_sum(qq[r]) / d + a.hd.eps);
  for (uint32_t c = lane; c < d; c += 64) {
    const bool first = c == lane;
    const float gg = first ? gg0 : a.ln_g[c], bb = first ? bb0 : a.ln_b[c];
#pragma unroll
    for (uint32_t r = 0; r < kRowsPerWave; ++r) {
      float v = (xs[wave * kRowsPerWave + r][c] - s[r]) * qq[r] * gg + bb;
      if (!FRONT) v *= first ? gate0[r] : a.gate[static_cast<uint64_t>(row[r]) * d + c];
      xs[wave * kRowsPerWave + r][c] = v;
    }
  }
  __builtin_amdgcn_wave_barrier();
  float acc[kRowsPerWave][4];  // four partial sums: shorter dependence chains and rounding errors
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0f;
  for (uint32_t k0 = 0; k0 < d; k0 += kAhead) {
    float wn[kAhead];
    const uint32_t next = k0 + kAhead < d ? k0 + kAhead : 0;
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) wn[k] = wc[static_cast<uint64_t>(next + k) * a.n_out];
#pragma unroll
    for (uint32_t r = 0; r < kRowsPerWave; ++r) {
      const float4* xr = reinterpret_cast<const float4*>(&xs[wave * kRowsPerWave + r][k0]);
#pragma unroll
      for (uint32_t k = 0; k < kAhead / 4; ++k) {
        const float4 x = xr[k];
        acc[r][0] = fmaf(x.x, wr[4 * k], acc[r][0]);
        acc[r][1] = fmaf(x.y, wr[4 * k + 1], acc[r][1]);
        acc[r][2] = fmaf(x.z, wr[4 * k + 2], acc[r][2]);
        acc[r][3] = fmaf(x.w, wr[4 * k + 3], acc[r][3]);
      }
    }
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) wr[k] = wn[k];
  }
  if (!col_ok) return;
#pragma unroll
  for (uint32_t r = 0; r < kRowsPerWave; ++r) {
    if (row0 + r >= a.N) continue;
    const float sum = (acc[r][0] + acc[r][1]) + (acc[r][2] + acc[r][3]);
    if (!FRONT) {
      a.y[static_cast<uint64_t>(row[r]) * d + col] = resid[r] + sum + bias;
      continue;
    }
    const float z = silu(sum + bias);
    if ((which & 1) == 0) {
      (which == 0 ? a.u : a.q)[static_cast<uint64_t>(row[r]) * d + c_out] = z;
      continue;
    }
    if (page[r] < 0 || static_cast<uint32_t>(page[r]) >= a.kv.n_pages) {
      if (c_out == 0) atomicAdd(&a.kv.counters[ctr_index(kCtrBadPages)], 1ull);
      continue;
    }
    const uint32_t head = c_out / a.hd.dh, cc = c_out % a.hd.dh;
    float* blk = reinterpret_cast<float*>(a.kv.base + static_cast<uint64_t>(page[r]) * a.kv.page_size + kv_block_offset(a.hd, a.layer, which == 1 ? 1 : 0, head, 4));
    if (which == 3) blk[static_cast<uint64_t>(tok[r]) * a.hd.dh + cc] = z;  // K: [token][d_h]
    else blk[static_cast<uint64_t>(cc) * a.hd.pt + tok[r]] = z;             // V: [d_h][token]
  }
}

// ---------------------------------------------------------------------------------------
// Paged attention: one block per (16 queries of one request, head), d_h <= 16 * NS.  The wavefronts take groups of 16
// keys in turn and add their sums at the end; nothing is shared before that, so there is no barrier in the loop and a
// wavefront's loads for the next group fly during the current one.  Both products run on v_mfma_f32_16x16x4_f32 (full
// fp32 multiply-adds): S^T = K Q^T leaves a lane with one query (lane % 16) and the four keys 4 * (lane / 16) + r; these
// are, step r for register r, the second operand of O^T += V^T P^T, whose first operand is then four consecutive keys of
// one row of V^T: one 16-byte load straight from the page, as K's are (which elements of d_h a step contracts over does not
// matter as long as K and Q agree: lane group g takes 16 s + 4 g .. + 4).
// 4 requests x 256 tokens, 2 heads: 10.4 us (one wavefront per query and head, whose lanes fetched whole rows of K and V on
// their own, 71 us; 16-query blocks on tiles staged in LDS, 22 us).
// ---------------------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
static_assert(kF32Queries == 16, "one MFMA tile of queries");

template <int NS, uint32_t WAVES>
__global__ __launch_bounds__(64 * WAVES) void attention_f32(HstuDims hd, uint32_t layer, const float* __restrict__ q,
                                                     const float* __restrict__ pos, const float* __restrict__ time,
                                                     KvView kv, const ReqDev* __restrict__ reqs,
                                                     const F32Tile* __restrict__ tiles, const int32_t* __restrict__ page_tables,
                                                     const long long* __restrict__ ts, float* __restrict__ o) {
  __shared__ __attribute__((aligned(16))) f32x4 sums[WAVES - 1][NS][64];
  __shared__ float times[64];
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, li = lane & 15, h = blockIdx.y;
  const F32Tile tile = tiles[blockIdx.x];
  const ReqDev rq = reqs[tile.req];
  const uint32_t q0 = tile.q0;  // first query of the tile among the request's new tokens
  const uint32_t nq = rq.new_len - q0 < 16 ? rq.new_len - q0 : 16;
  const bool ok = li < nq;
  const uint32_t dh = hd.dh;
  const bool vec = (dh & 3) == 0 && (hd.pt & 3) == 0;  // 16-byte loads are aligned and stay inside a row and a page
  const uint32_t last = rq.prefix_len + q0 + nq - 1;
  const uint32_t p = rq.prefix_len + q0 + (ok ? li : 0);
  const long long* tsr = ts + rq.ts_off;
  const float* pos_h = pos + (static_cast<uint64_t>(layer) * hd.H + h) * hd.n_pos;
  const uint64_t koff = kv_block_offset(hd, layer, 0, h, 4), voff = kv_block_offset(hd, layer, 1, h, 4);
  if (tid < 64) times[tid] = tid < hd.n_time ? time[(static_cast<uint64_t>(layer) * hd.H + h) * hd.n_time + tid] : 0.0f;
  const long long ts_p = tsr[p];
  // four elements from c on of a row of d_h elements
  auto row4 = [&](const float* row, uint32_t c) {
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (vec && c < dh) return *reinterpret_cast<const f32x4*>(row + c);
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e)
      if (c + e < dh) v[e] = row[c + e];
    return v;
  };
  f32x4 qf[NS], acc[NS];
#pragma unroll
  for (uint32_t s = 0; s < NS; ++s) {
    qf[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    acc[s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if (ok) qf[s] = row4(q + static_cast<uint64_t>(rq.x_off + q0 + li) * hd.d + h * dh, 16 * s + 4 * g);
  }
  auto page_at = [&](uint32_t j, uint32_t* tok) -> const uint8_t* {
    uint32_t pi;
    split_token(hd, j, &pi, tok);
    const int32_t page = page_tables[rq.page_table_off + pi];
    return page >= 0 && static_cast<uint32_t>(page) < kv.n_pages ? kv.base + static_cast<uint64_t>(page) * kv.page_size : nullptr;
  };
  struct Group {  // of 16 keys: this lane's operands, key times and positional biases
    f32x4 k[NS], v[NS];
    long long t[4];
    float bias[4];
  };
  auto fetch = [&](uint32_t j0, Group& b) {
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t tok = 0;
    const uint8_t* pb = j0 + li <= last ? page_at(j0 + li, &tok) : nullptr;
    if (!pb && j0 + li <= last && g == 0) atomicAdd(&kv.counters[ctr_index(kCtrBadPages)], 1ull);
#pragma unroll
    for (uint32_t s = 0; s < NS; ++s)  // row li of K
      b.k[s] = pb ? row4(reinterpret_cast<const float*>(pb + koff) + static_cast<uint64_t>(tok) * dh, 16 * s + 4 * g) : zero;
    const uint32_t jv = j0 + 4 * g;  // keys jv .. jv + 3 of rows 16 s + li of V^T
    if (vec && jv + 3 <= last) {
      pb = page_at(jv, &tok);
#pragma unroll
      for (uint32_t s = 0; s < NS; ++s)
        b.v[s] = pb && 16 * s + li < dh
                     ? *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(pb + voff) + static_cast<uint64_t>(16 * s + li) * hd.pt + tok)
                     : zero;
    } else {
#pragma unroll
      for (uint32_t s = 0; s < NS; ++s) b.v[s] = zero;
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) {
        if (jv + e > last) continue;
        pb = page_at(jv + e, &tok);
#pragma unroll
        for (uint32_t s = 0; s < NS; ++s)
          if (pb && 16 * s + li < dh) b.v[s][e] = reinterpret_cast<const float*>(pb + voff)[static_cast<uint64_t>(16 * s + li) * hd.pt + tok];
      }
    }
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) {
      const uint32_t j = jv + e, rel = j > p ? 0 : (p - j < hd.n_pos - 1 ? p - j : hd.n_pos - 1);
      b.t[e] = tsr[j <= last ? j : last];
      b.bias[e] = pos_h[rel];
    }
  };
  // In the product a key that a query does not see counts with probability 0, which would still spoil the query's sum if
  // the key's values are infinite or not numbers.  Such values are taken out here and added to the queries that see them.
  auto take_out_odd = [&](f32x4 (&v)[NS], const f32x4& pr, uint32_t j0) {
#pragma unroll
    for (uint32_t s = 0; s < NS; ++s) {
      f32x4 rest, is_odd;
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) {
        const bool odd = v[s][e] * 0.0f != 0.0f;
        rest[e] = odd ? v[s][e] : 0.0f;
        is_odd[e] = odd ? 1.0f : 0.0f;
        v[s][e] = odd ? 0.0f : v[s][e];
      }
#pragma unroll 1
      for (uint32_t key = 0; key < 16; ++key) {
        auto pick = [&](const f32x4& x) { return g == key / 4 ? (key & 2 ? (key & 1 ? x[3] : x[2]) : (key & 1 ? x[1] : x[0])) : 0.0f; };
        const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
        const f32x4 part = __builtin_amdgcn_mfma_f32_16x16x4f32(pick(rest), pick(pr), zero, 0, 0, 0);
        const f32x4 here = __builtin_amdgcn_mfma_f32_16x16x4f32(pick(is_odd), 1.0f, zero, 0, 0, 0);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r)
          if (here[r] != 0.0f && j0 + key <= p) acc[s][r] += part[r];
      }
    }
  };
  const uint32_t n_groups = last / 16 + 1;
  Group cur, next;
  if (wave < n_groups) fetch(16 * wave, cur);
  __syncthreads();  // times is there
  for (uint32_t k = wave; k < n_groups; k += WAVES) {
    if (k + WAVES < n_groups) fetch(16 * (k + WAVES), next);
    f32x4 s4 = {cur.bias[0], cur.bias[1], cur.bias[2], cur.bias[3]};
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) s4[e] += times[time_bucket(ts_p - cur.t[e], hd.n_time)];
#pragma unroll
    for (uint32_t s = 0; s < NS; ++s)
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) s4 = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.k[s][e], qf[s][e], s4, 0, 0, 0);
    f32x4 pr;
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e) pr[e] = 16 * k + 4 * g + e <= p ? s4[e] / (1.0f + expf(-s4[e])) : 0.0f;
    if (16 * k + 15 > rq.prefix_len + q0) {  // some query may not see some key
      float odd = 0.0f;                      // stays 0 unless a value is infinite or not a number
#pragma unroll
      for (uint32_t s = 0; s < NS; ++s)
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) odd += cur.v[s][e] * 0.0f;
      if (__any(odd != 0.0f)) take_out_odd(cur.v, pr, 16 * k);
    }
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e)
#pragma unroll
      for (uint32_t s = 0; s < NS; ++s) acc[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.v[s][e], pr[e], acc[s], 0, 0, 0);
    cur = next;
  }
  if (wave) {
#pragma unroll
    for (uint32_t s = 0; s < NS; ++s) sums[wave - 1][s][lane] = acc[s];
  }
  __syncthreads();
  if (wave || !ok) return;
  // acc[s][r]: element 16 s + 4 g + r of query li
#pragma unroll
  for (uint32_t s = 0; s < NS; ++s) {
#pragma unroll
    for (uint32_t w = 0; w < WAVES - 1; ++w) acc[s] += sums[w][s][lane];
    float* dst = o + static_cast<uint64_t>(rq.x_off + q0 + li) * hd.d + h * dh;
#pragma unroll
    for (uint32_t e = 0; e < 4; ++e)
      if (16 * s + 4 * g + e < dh) dst[16 * s + 4 * g + e] = acc[s][e] * hd.inv_n;
  }
}

}  // namespace

hipError_t launch_layer_half_f32(const HstuDims& hd, uint32_t layer, bool front, const float* in, const float* gate, const float* ln_g,
                                 const float* ln_b, const float* w, const float* bias, float* u, float* q, const KvView& kv,
                                 const StepLists& sl, const int32_t* page_tables, const float* resid, float* y, hipStream_t stream) {
  if (sl.N == 0) return hipSuccess;
  if (hd.d > kMaxWidth || hd.d % kAhead != 0) return hipErrorInvalidValue;
  HalfArgsF32 a{hd, layer, sl.N, sl.B, front ? 4 * hd.d : hd.d, in, gate, ln_g, ln_b, w, bias, u, q, kv, sl.reqs, page_tables, resid, y};
  const dim3 grid((sl.N + kRowsPerBlock - 1) / kRowsPerBlock, (a.n_out + 63) / 64), block(256);
  if (front) hipLaunchKernelGGL(layer_half_f32<true>, grid, block, 0, stream, a);
  else hipLaunchKernelGGL(layer_half_f32<false>, grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_attention_f32(const HstuDims& hd, uint32_t layer, const float* q, const float* pos, const float* time, const KvView& kv,
                                const StepLists& sl, const int32_t* page_tables, const int64_t* ts, float* o, hipStream_t stream) {
  if (sl.n_f32_tiles == 0) return hipSuccess;
  if (hd.dh > 64) return hipErrorInvalidValue;
  const dim3 grid(sl.n_f32_tiles, hd.H);
  const long long* t = reinterpret_cast<const long long*>(ts);
  const uint32_t waves = f32_waves(hd.dh, static_cast<uint64_t>(sl.n_f32_tiles) * hd.H, sl.longest, sl.f32_keys / sl.n_f32_tiles);
  auto run = [&](auto kernel, uint32_t w) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * w), 0, stream, hd, layer, q, pos, time, kv, sl.reqs, sl.f32_tiles, page_tables, t, o);
  };
  switch ((hd.dh + 15) / 16) {
#define RACER_F32_CASE(S, MOST)                                    \
  case S:                                                          \
    if (waves == 4) run(attention_f32<S, 4>, 4);                   \
    else if (waves == 8 || MOST == 8) run(attention_f32<S, 8>, 8); \
    else run(attention_f32<S, MOST>, MOST);                        \
    break;
    RACER_F32_CASE(1, 16) RACER_F32_CASE(2, 16) RACER_F32_CASE(3, 8) RACER_F32_CASE(4, 8)
#undef RACER_F32_CASE
  }
  return hipGetLastError();
}

}  // namespace racer
