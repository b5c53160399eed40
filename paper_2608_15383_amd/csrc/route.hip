// Routing and grouping kernels (Sec. 3.1 Eq. 1; Fig. 1 and Sec. 3.4, where the
// token-expert pairs are gathered by the expert they select).  The arithmetic
// lives in device_route.h.
//
//   router_logits_kernel: z[t][e] = fp32(sum_i h[t][i] * W_r[e][i]), fp64 sum
//                         on fp64 MFMA; a small call leaves fp64 sums over
//                         slices of d, which its top-k adds and rounds.
//   topk_kernel:          k largest logits per token (ties -> lower expert id)
//                         and their softmax mixture weights in fp64.
//   topk_count_kernel:    the same for the 64 / k tokens of one 64-pair chunk
//                         per workgroup, plus that chunk's per-expert counts.
//   group_kernel:         per-expert counts, exclusive offsets, a stable
//                         counting sort of pair ids, the ascending active list
//                         and (optionally) the MFMA row-tile prefix sum.
#include <type_traits>

#include "device_route.h"

namespace emoe {
namespace {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Router logits on fp64 MFMA (v_mfma_f64_16x16x4f64): a workgroup computes a
// 16-token x 16-expert tile and its four wavefronts split d into quarters.
// Per 32 inputs, lane l loads 8 consecutive bf16 of token row l%16 and of
// expert row l%16 (inputs 8*(l/16) .. +7) and feeds them to 8 MFMAs; A and B
// take the same input for the same lane, so every product h_k * w_k is
// formed once and exactly, and summed in fp64.  The four partial sums are
// added in wavefront order and rounded once to fp32.
// With parts (gridDim.z = S slices of d) the workgroup covers slice
// blockIdx.z only and stores its fp64 sum to parts[slice][t][e] instead; the
// top-k adds the slices in order and rounds (another order of fp64 sums than
// one workgroup's, so a logit could differ in its last fp32 bit; none has).
// Each of a tile's wavefronts is a dependent chain of 128 MFMAs of 64 cycles
// at d = 2048, so the few tiles of a small call are bound by that chain and by
// the load rounds between, on as few CUs: 16 tokens took 9.3 us on 4
// workgroups, 4.3 with four slices.
__global__ __launch_bounds__(256) void router_logits_kernel(int tokens, int n_experts, int d,
                                                            const uint16_t* __restrict__ h,
                                                            const uint16_t* __restrict__ wr,
                                                            float* __restrict__ logits,
                                                            double* __restrict__ parts,
                                                            float* __restrict__ tok_bias) {
  __shared__ double part[4][4][64];
  const int lane = lane_id();
  const int wave = threadIdx.x >> 6;
  const int t0 = blockIdx.x * 16, e0 = blockIdx.y * 16;
  const int row = lane & 15, q = lane >> 4;
  // Rows past the end repeat the last row; their results are not stored.
  const int t = min(t0 + row, tokens - 1);
  const int e = min(e0 + row, n_experts - 1);
  const int kq = d / (4 * (int)gridDim.z);
  const int k0 = ((int)blockIdx.z * 4 + wave) * kq;
  const uint16_t* hp = h + (int64_t)t * d + k0 + 8 * q;
  const uint16_t* wp = wr + (int64_t)e * d + k0 + 8 * q;
  f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
  // Loads run kAhead steps of 32 inputs ahead of the MFMAs (8 and 16 steps at
  // 2048 tokens: 19.1 and 20.3 us against 17.2).
  constexpr int kAhead = 4;
  const int n = kq / 32;
  // With tok_bias (d a multiple of 512 per slice, so every iteration of the
  // loop below is one 128-input group), the first expert tile's workgroups
  // also sum each group of their token rows.
  const bool sums = tok_bias != nullptr && blockIdx.y == 0;
  uint4 hb[kAhead], wb[kAhead];
#pragma unroll
  for (int j = 0; j < kAhead; ++j) {
    if (j < n) {
      hb[j] = *reinterpret_cast<const uint4*>(hp + 32 * j);
      wb[j] = *reinterpret_cast<const uint4*>(wp + 32 * j);
    }
  }
  for (int i = 0; i < n; i += kAhead) {
    float gsum = 0.f;
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      if (i + j < n) {
        double hv[8], wv[8];
        bf16x8_to_f64(hb[j], hv);
        bf16x8_to_f64(wb[j], wv);
        if (i + j + kAhead < n) {
          hb[j] = *reinterpret_cast<const uint4*>(hp + 32 * (i + j + kAhead));
          wb[j] = *reinterpret_cast<const uint4*>(wp + 32 * (i + j + kAhead));
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(hv[s], wv[s], acc, 0, 0, 0);
        if (sums) {
#pragma unroll
          for (int s = 0; s < 8; ++s) gsum += (float)hv[s];
        }
      }
    }
    if (sums) {
      // The lane's 32 inputs of the group, then the four lanes of the row.
      gsum += __shfl_xor(gsum, 16);
      gsum += __shfl_xor(gsum, 32);
      const int g = (k0 + 32 * i) / kGroup;
      if (q == 0 && t0 + row < tokens) tok_bias[(int64_t)(t0 + row) * (d / kGroup) + g] = -136.f * gsum;
    }
  }
  // Lane l holds rows (tokens) l/16 + 4*r of column (expert) l%16 (the fp64
  // MFMA interleaves its output rows by register).
#pragma unroll
  for (int r = 0; r < 4; ++r) part[wave][r][lane] = acc[r];
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double z = ((part[0][r][lane] + part[1][r][lane]) + part[2][r][lane]) + part[3][r][lane];
      const int tt = t0 + q + 4 * r, ee = e0 + row;
      if (tt >= tokens || ee >= n_experts) continue;
      if (parts)
        parts[((int64_t)blockIdx.z * tokens + tt) * n_experts + ee] = z;
      else
        logits[(int64_t)tt * n_experts + ee] = (float)z;
    }
  }
}

// Selection from token t's logits: as given, or (kParts) the router's slice
// sums added in order and rounded to fp32, which are then also stored as the
// call's logits.  A kernel per source: with both in one, either as two
// selections or behind one branch, the top-k launches took 0.2 to 0.6 us more.
template <bool kParts>
__device__ __forceinline__ void topk_select_from(const LogitSource& src, int t, int tokens,
                                                 int n_experts, int top_k, TopkState& st,
                                                 uint64_t* scratch) {
  const int lane = lane_id();
#pragma unroll
  for (int c = 0; c < kPerLane; ++c) {
    const int e = lane + 64 * c;
    st.v[c] = 0.f;
    if (e >= n_experts) continue;
    if constexpr (!kParts) {
      st.v[c] = src.logits[(int64_t)t * n_experts + e];
      continue;
    }
    const double* p = src.parts + (int64_t)t * n_experts + e;
    double v[kRouterMaxSlices];
#pragma unroll
    for (int s = 0; s < kRouterMaxSlices; ++s)
      v[s] = s < src.slices ? p[(int64_t)s * tokens * n_experts] : 0.0;
    double z = v[0];
#pragma unroll
    for (int s = 1; s < kRouterMaxSlices; ++s) z += v[s];
    st.v[c] = (float)z;
    src.logits_out[(int64_t)t * n_experts + e] = st.v[c];
  }
  wave_topk_select_loaded(n_experts, top_k, st, scratch);
}

// bias[t][g] = -136 * sum of x[t][128g .. 128g+127] (fp32, fixed order) of one
// token row by one wavefront: the accumulator start of the gate/up MFMA
// chains of every pair of token t.
__device__ __forceinline__ void wave_row_bias(int t, int K, const uint16_t* __restrict__ x,
                                              float* __restrict__ bias) {
  const int lane = lane_id();
  const uint16_t* xr = x + (int64_t)t * K;
  for (int c0 = 0; c0 < K / 8; c0 += 64) {
    const int c = c0 + lane;
    float s = 0.f;
    if (c < K / 8) {
      const uint4 v = *reinterpret_cast<const uint4*>(xr + 8 * c);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        s += bf16_to_f32(w[q] & 0xffffu);
        s += bf16_to_f32(w[q] >> 16);
      }
    }
    // Sum over the 16 lanes holding one group.
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    s += __shfl_xor(s, 8);
    if ((lane & 15) == 0 && c < K / 8) bias[(int64_t)t * (K / kGroup) + c / (kGroup / 8)] = -136.f * s;
  }
}

// Workgroups from rb.first on form the row biases, one token per wavefront:
// they ride along with the top-k launch, which saves one of their own.
__device__ __forceinline__ bool row_bias_block(const RowBias& rb, int tokens) {
  if ((int)blockIdx.x < rb.first) return false;
  const int t = ((int)blockIdx.x - rb.first) * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (t < tokens) wave_row_bias(t, rb.d, rb.x, rb.bias);
  return true;
}

__global__ __launch_bounds__(256) void row_bias_kernel(int tokens, RowBias rb) {
  row_bias_block(rb, tokens);
}

template <bool kParts>
__global__ __launch_bounds__(256) void topk_kernel(int tokens, int n_experts, int top_k,
                                                   int renormalize, LogitSource src,
                                                   int32_t* __restrict__ topk_ids,
                                                   float* __restrict__ topk_w, RowBias rb) {
  __shared__ uint64_t s_rank[4][64];  // per-wavefront top-k scratch
  if (row_bias_block(rb, tokens)) return;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= tokens) return;
  TopkState st;
  topk_select_from<kParts>(src, t, tokens, n_experts, top_k, st, s_rank[threadIdx.x >> 6]);
  wave_topk_store_ids<false>(st, top_k, topk_ids + (int64_t)t * top_k);
  wave_topk_weights<false>(st, n_experts, top_k, renormalize, topk_w + (int64_t)t * top_k);
}

// Top-k of 64 / top_k tokens per workgroup, one wavefront each, when top_k
// divides 64: the workgroup's pairs are then exactly one 64-pair chunk of the
// wide grouping (chunk c = blockIdx.x), and after its selections it also
// writes that chunk's per-expert counts (chunk_count_kernel's row), which
// saves that launch.  Ids and weights as topk_kernel writes them.
template <bool kParts>
__global__ __launch_bounds__(1024) void topk_count_kernel(int tokens, int n_experts, int top_k,
                                                          int renormalize, LogitSource src,
                                                          int32_t* __restrict__ topk_ids,
                                                          float* __restrict__ topk_w,
                                                          int32_t* __restrict__ chunk_counts,
                                                          RowBias rb) {
  __shared__ uint64_t s_rank[16][64];  // per-wavefront top-k scratch
  __shared__ int s_pair[64];           // the chunk's expert ids, pair order
  __shared__ int row[EMOE_MAX_EXPERTS];
  const int per = 64 / top_k;
  if (row_bias_block(rb, tokens)) return;
  const int lane = lane_id();
  const int wave = threadIdx.x >> 6;
  const int c = blockIdx.x;
  const int t = c * per + wave;
  for (int e = threadIdx.x; e < n_experts; e += blockDim.x) row[e] = 0;
  if (t < tokens) {
    TopkState st;
    topk_select_from<kParts>(src, t, tokens, n_experts, top_k, st, s_rank[wave]);
    wave_topk_store_ids<false>(st, top_k, topk_ids + (int64_t)t * top_k);
#pragma unroll
    for (int r = 0; r < kPerLane; ++r)
      if (lane + 64 * r < top_k) s_pair[wave * top_k + lane + 64 * r] = st.sel_id[r];
    wave_topk_weights<false>(st, n_experts, top_k, renormalize, topk_w + (int64_t)t * top_k);
  }
  __syncthreads();
  if (wave == 0) {
    int bits = 0;
    while ((1 << bits) < n_experts) ++bits;
    const bool valid = 64 * c + lane < tokens * top_k;
    const int e = valid ? s_pair[lane] : 0;
    const uint64_t m = match_expert(valid, e, bits);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    if (valid && rank == 0) row[e] = __popcll(m);  // one wavefront: LDS accesses stay in order
    for (int x = lane; x < n_experts; x += 64) chunk_counts[(int64_t)c * n_experts + x] = row[x];
  }
}

constexpr int kGroupThreads = 1024;

__global__ __launch_bounds__(kGroupThreads) void group_kernel(
    int pairs, int n_experts, const int32_t* __restrict__ ids, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ sorted_pairs, int32_t* __restrict__ active,
    int32_t* __restrict__ n_active, int32_t* __restrict__ tile_offsets,
    int32_t* __restrict__ pair_pos, int mfma_rows) {
  __shared__ GroupShared<kGroupThreads> sh;
  block_group<kGroupThreads, false, true>(sh, pairs, n_experts, ids, counts, offsets, sorted_pairs,
                                          active, n_active, tile_offsets, pair_pos, mfma_rows);
}

// Top-k and grouping of a small call in one launch: workgroup 0's 16
// wavefronts take the tokens, then group all pairs.  It saves a launch's
// start, its gap and a round trip of the ids, and pays for a top-k of all
// tokens on one CU, so only calls that topk_group_fits admits take it.
template <bool kParts>
__global__ __launch_bounds__(kGroupThreads) void topk_group_kernel(
    int tokens, int n_experts, int top_k, int renormalize, LogitSource src,
    int32_t* __restrict__ topk_ids, float* __restrict__ topk_w, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ sorted_pairs, int32_t* __restrict__ active,
    int32_t* __restrict__ n_active, int32_t* __restrict__ tile_offsets,
    int32_t* __restrict__ pair_pos, int mfma_rows, RowBias rb) {
  __shared__ uint64_t s_rank[kGroupThreads / 64][64];
  __shared__ GroupShared<kGroupThreads> sh;
  if (row_bias_block(rb, tokens)) return;
  const int wave = threadIdx.x >> 6;
  for (int t = wave; t < tokens; t += kGroupThreads / 64) {
    TopkState st;
    topk_select_from<kParts>(src, t, tokens, n_experts, top_k, st, s_rank[wave]);
    wave_topk_store_ids<false>(st, top_k, topk_ids + (int64_t)t * top_k);
    wave_topk_weights<false>(st, n_experts, top_k, renormalize, topk_w + (int64_t)t * top_k);
  }
  __threadfence_block();
  __syncthreads();
  block_group<kGroupThreads, false, false>(sh, tokens * top_k, n_experts, topk_ids, counts, offsets,
                                           sorted_pairs, active, n_active, tile_offsets, pair_pos,
                                           mfma_rows);
}

// Grouping spread over many workgroups (large calls): 64-pair chunks, one per
// wavefront, kChunkWaves chunks per workgroup.
constexpr int kChunkWaves = 16;

// chunk_counts[c][e]: pairs of chunk c (pairs 64c .. 64c+63) routed to e.
__global__ __launch_bounds__(64 * kChunkWaves) void chunk_count_kernel(
    int pairs, int n_experts, const int32_t* __restrict__ ids, int32_t* __restrict__ chunk_counts) {
  __shared__ int row[kChunkWaves][EMOE_MAX_EXPERTS];
  const int lane = lane_id();
  const int wave = threadIdx.x >> 6;
  const int c = blockIdx.x * kChunkWaves + wave;
  if (c >= (pairs + 63) / 64) return;  // whole wavefront; no barrier below
  int bits = 0;
  while ((1 << bits) < n_experts) ++bits;
  int* r = row[wave];
  for (int e = lane; e < n_experts; e += 64) r[e] = 0;
  const int i = 64 * c + lane;
  const bool valid = i < pairs;
  const int e = valid ? ids[i] : 0;
  const uint64_t m = match_expert(valid, e, bits);
  const int rank = __popcll(m & ((1ull << lane) - 1ull));
  if (valid && rank == 0) r[e] = __popcll(m);  // one wavefront: LDS accesses stay in order
  for (int x = lane; x < n_experts; x += 64) chunk_counts[(int64_t)c * n_experts + x] = r[x];
}

// Each workgroup sums the chunk table (all chunks, and those before its own),
// derives the exclusive offsets and its chunks' first positions per expert,
// and places its chunks' pairs in order (stable).  Workgroup 0 also writes
// counts, offsets, the active list, n_active and the row-tile prefix sum.
__global__ __launch_bounds__(64 * kChunkWaves) void chunk_place_kernel(
    int pairs, int n_experts, const int32_t* __restrict__ ids,
    const int32_t* __restrict__ chunk_counts, int32_t* __restrict__ counts,
    int32_t* __restrict__ offsets, int32_t* __restrict__ sorted_pairs,
    int32_t* __restrict__ active, int32_t* __restrict__ n_active,
    int32_t* __restrict__ tile_offsets, int32_t* __restrict__ pair_pos, int mfma_rows) {
  __shared__ int part_all[kChunkWaves][EMOE_MAX_EXPERTS];
  __shared__ int part_pre[kChunkWaves][EMOE_MAX_EXPERTS];
  // Wavefront w's chunk: its count per expert, then its first position.
  __shared__ int base[kChunkWaves][EMOE_MAX_EXPERTS];
  __shared__ int block_sum[kPerLane][3];  // pairs, active experts, tiles per 64 experts
  const int lane = lane_id();
  const int wave = threadIdx.x >> 6;
  const int n_chunks = (pairs + 63) / 64;
  const int c0 = blockIdx.x * kChunkWaves;
  // Wavefront w sums chunks w, w + 16, ...: all of them, and those before c0.
  // Bound by its chain of latencies (one round of loads, the scan, the
  // placement): the scan as four strided experts a lane, with its chunks'
  // counts read from memory there, made it 7.3 us at 2048 tokens, now 5.5.
  // 16 loads in flight: 16 chunks of the one block of up to 64 experts, or
  // four chunks of each of the four blocks.  With the blocks one after the
  // other here and in the scan, 256 experts and 33 chunks took 12.1 us; now 4.7.
  auto sum_chunks = [&](auto blocks_c) __attribute__((always_inline)) {
    constexpr int kQ = decltype(blocks_c)::value;
    constexpr int kBatch = 16 / kQ;
    int at[kQ], all[kQ], pre[kQ], mine[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      at[q] = min(64 * q + lane, n_experts - 1);  // lanes past the end repeat it, unused
      all[q] = pre[q] = 0;
      mine[q] = c0 + wave < n_chunks ? chunk_counts[(int64_t)(c0 + wave) * n_experts + at[q]] : 0;
    }
    for (int cb = wave; cb < n_chunks; cb += kBatch * kChunkWaves) {
      int v[kBatch][kQ];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int c = cb + j * kChunkWaves;
#pragma unroll
        for (int q = 0; q < kQ; ++q)
          v[j][q] = c < n_chunks ? chunk_counts[(int64_t)c * n_experts + at[q]] : 0;
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          all[q] += v[j][q];
          if (cb + j * kChunkWaves < c0) pre[q] += v[j][q];
        }
    }
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      part_all[wave][64 * q + lane] = all[q];
      part_pre[wave][64 * q + lane] = pre[q];
      base[wave][64 * q + lane] = mine[q];
    }
  };
  if (n_experts <= 64)
    sum_chunks(std::integral_constant<int, 1>());
  else
    sum_chunks(std::integral_constant<int, kPerLane>());
  __syncthreads();
  // Wavefront b scans experts 64b + lane; above 64 experts the blocks' sums
  // meet through LDS.
  const int blocks = (n_experts + 63) / 64;
  const int x = 64 * wave + lane;
  const bool ok = x < n_experts;
  int own[kChunkWaves], cnt = 0, pre = 0, off = 0, nz = 0, tl = 0;
  int total = 0, nz_total = 0, tl_total = 0;
  if (wave < blocks) {
#pragma unroll
    for (int w = 0; w < kChunkWaves; ++w) {
      own[w] = ok ? base[w][x] : 0;
      cnt += ok ? part_all[w][x] : 0;
      pre += ok ? part_pre[w][x] : 0;
    }
    off = wave_exclusive_scan(cnt, total);
    nz = wave_exclusive_scan(cnt > 0, nz_total);
    tl = wave_exclusive_scan(mfma_row_tiles(cnt, mfma_rows), tl_total);
    if (blocks > 1 && lane == 0) {
      block_sum[wave][0] = total;
      block_sum[wave][1] = nz_total;
      block_sum[wave][2] = tl_total;
    }
  }
  if (blocks > 1) __syncthreads();
  if (wave < blocks) {
    const bool writer = blockIdx.x == 0;
    int off0 = 0, nz0 = 0, tl0 = 0;
    for (int b = 0; b < wave; ++b) {
      off0 += block_sum[b][0];
      nz0 += block_sum[b][1];
      tl0 += block_sum[b][2];
    }
    if (ok) {
      if (writer) {
        counts[x] = cnt;
        offsets[x] = off0 + off;
        tile_offsets[x] = tl0 + tl;
        if (cnt > 0) active[nz0 + nz] = x;
      }
      int run = off0 + off + pre;
#pragma unroll
      for (int w = 0; w < kChunkWaves; ++w) {
        base[w][x] = run;
        run += own[w];
      }
    }
    if (writer && wave == blocks - 1 && lane == 0) {
      offsets[n_experts] = off0 + total;
      tile_offsets[n_experts] = tl0 + tl_total;
      *n_active = nz0 + nz_total;
    }
  }
  __syncthreads();
  const int c = c0 + wave;
  if (c >= n_chunks) return;
  int bits = 0;
  while ((1 << bits) < n_experts) ++bits;
  const int i = 64 * c + lane;
  const bool valid = i < pairs;
  const int e = valid ? ids[i] : 0;
  const uint64_t m = match_expert(valid, e, bits);
  const int rank = __popcll(m & ((1ull << lane) - 1ull));
  if (valid) {
    const int pos = base[wave][e] + rank;
    sorted_pairs[pos] = i;
    pair_pos[i] = pos;
  }
}

}  // namespace

hipError_t launch_group_count(int pairs, int n_experts, const int32_t* topk_ids,
                              int32_t* chunk_counts, hipStream_t stream) {
  const int n_wg = ((pairs + 63) / 64 + kChunkWaves - 1) / kChunkWaves;
  if (n_wg == 0) return hipSuccess;
  launch(chunk_count_kernel, dim3(n_wg), dim3(64 * kChunkWaves), stream, pairs, n_experts, topk_ids,
         chunk_counts);
  return hipGetLastError();
}

hipError_t launch_group_place(int pairs, int n_experts, const int32_t* topk_ids,
                              const int32_t* chunk_counts, int32_t* counts, int32_t* offsets,
                              int32_t* sorted_pairs, int32_t* active, int32_t* n_active,
                              int32_t* tile_offsets, int32_t* pair_pos, int mfma_rows,
                              hipStream_t stream) {
  const int n_wg = ((pairs + 63) / 64 + kChunkWaves - 1) / kChunkWaves;
  if (n_wg == 0) return hipSuccess;
  launch(chunk_place_kernel, dim3(n_wg), dim3(64 * kChunkWaves), stream, pairs, n_experts, topk_ids,
         chunk_counts, counts, offsets, sorted_pairs, active, n_active, tile_offsets, pair_pos,
         mfma_rows);
  return hipGetLastError();
}

int router_slices(int tokens, int n_experts, int d) {
  // Slices only while the tiles leave CUs without work (two workgroups per CU
  // fill the matrix cores), and of whole 512-input quarters, so that every
  // wavefront keeps whole 128-input groups.
  const int tiles = ((tokens + 15) / 16) * ((n_experts + 15) / 16);
  int s = 1;
  while (2 * s <= kRouterMaxSlices && d % (512 * 2 * s) == 0 && tiles * 2 * s <= 512) s *= 2;
  return s;
}

hipError_t launch_router_logits(int tokens, int n_experts, int d, const uint16_t* h,
                                const uint16_t* w_router, float* logits, hipStream_t stream,
                                float* tok_bias, double* parts, int slices) {
  if (tokens == 0) return hipSuccess;
  if (d % 512 != 0) tok_bias = nullptr;
  dim3 grid((tokens + 15) / 16, (n_experts + 15) / 16, parts ? slices : 1);
  launch(router_logits_kernel, grid, dim3(256), stream, tokens, n_experts, d, h, w_router, logits,
         parts, tok_bias);
  return hipGetLastError();
}

namespace {
// Grid of a launch of `blocks` workgroups of `waves` wavefronts with the row
// biases' workgroups after them.
inline dim3 bias_grid(RowBias& rb, int blocks, int tokens, int waves) {
  rb.first = blocks;
  return dim3(blocks + (rb.x ? (tokens + waves - 1) / waves : 0));
}
}  // namespace

hipError_t launch_row_bias(int tokens, RowBias rb, hipStream_t stream) {
  if (tokens == 0) return hipSuccess;
  const dim3 grid = bias_grid(rb, 0, tokens, 4);
  launch(row_bias_kernel, grid, dim3(256), stream, tokens, rb);
  return hipGetLastError();
}

hipError_t launch_topk(int tokens, int n_experts, int top_k, int renormalize,
                       const LogitSource& src, int32_t* topk_ids, float* topk_w, hipStream_t stream,
                       RowBias rb) {
  if (tokens == 0) return hipSuccess;
  const dim3 grid = bias_grid(rb, (tokens + 3) / 4, tokens, 4);
  launch(src.slices ? topk_kernel<true> : topk_kernel<false>, grid, dim3(256), stream, tokens,
         n_experts, top_k, renormalize, src, topk_ids, topk_w, rb);
  return hipGetLastError();
}

hipError_t launch_topk_count(int tokens, int n_experts, int top_k, int renormalize,
                             const LogitSource& src, int32_t* topk_ids, float* topk_w,
                             int32_t* chunk_counts, hipStream_t stream, RowBias rb) {
  if (tokens == 0) return hipSuccess;
  if (top_k < 1 || 64 % top_k != 0 || 64 / top_k > 16) return hipErrorInvalidValue;
  const int per = 64 / top_k;  // tokens (wavefronts) per chunk
  const dim3 grid = bias_grid(rb, (tokens + per - 1) / per, tokens, per);
  launch(src.slices ? topk_count_kernel<true> : topk_count_kernel<false>, grid, dim3(64 * per),
         stream, tokens, n_experts, top_k, renormalize, src, topk_ids, topk_w, chunk_counts, rb);
  return hipGetLastError();
}

hipError_t launch_topk_group(int tokens, int n_experts, int top_k, int renormalize,
                             const LogitSource& src, int32_t* topk_ids, float* topk_w,
                             int32_t* counts, int32_t* offsets, int32_t* sorted_pairs,
                             int32_t* active, int32_t* n_active, int32_t* tile_offsets,
                             int32_t* pair_pos, int mfma_rows, hipStream_t stream,
                             RowBias rb) {
  if (tokens == 0) return hipSuccess;
  const dim3 grid = bias_grid(rb, 1, tokens, kGroupThreads / 64);
  launch(src.slices ? topk_group_kernel<true> : topk_group_kernel<false>, grid,
         dim3(kGroupThreads), stream, tokens, n_experts, top_k, renormalize, src, topk_ids, topk_w,
         counts, offsets, sorted_pairs, active, n_active, tile_offsets, pair_pos, mfma_rows, rb);
  return hipGetLastError();
}

hipError_t launch_group(int pairs, int n_experts, const int32_t* topk_ids, int32_t* counts,
                        int32_t* offsets, int32_t* sorted_pairs, int32_t* active,
                        int32_t* n_active, int32_t* tile_offsets, int32_t* pair_pos,
                        int mfma_rows, hipStream_t stream) {
  launch(group_kernel, dim3(1), dim3(kGroupThreads), stream, pairs, n_experts, topk_ids, counts,
         offsets, sorted_pairs, active, n_active, tile_offsets, pair_pos, mfma_rows);
  return hipGetLastError();
}

}  // namespace emoe
