// Mixture-of-experts FFN around the grouped tile GEMM: routing, grouping of (token, slot) pairs
// by expert, and the fixed-order combine.
//
//   router logits [rows, E] (fp32, from the GEMM)  ->  softmax over all experts, top-k by value
//   with ties to the lower index, weights renormalised to sum 1 (no shared expert, no capacity
//   limit).  Every (token, slot) pair takes a place in its expert's group through an integer
//   atomic counter in LDS (one workgroup groups all pairs; device-scope atomics from every routing
//   wavefront on E addresses cost 25-40 us per launch); the order inside a group depends on
//   scheduling, but every pair's result is computed from its own row only and written to its own
//   (token, slot) row, and the combine adds the k slots of a token in slot order, so the output is
//   deterministic.
#include "s2d2_internal.h"
#include "../../include/s2d2.h"

namespace s2d2 {

static constexpr int MOE_MAX_E = 256;   // experts per lane <= 4

// One wavefront per row.
__global__ __launch_bounds__(256) void moe_route_kernel(const float* __restrict__ logits, int E, int top_k,
                                                        const int32_t* __restrict__ m_count,
                                                        int32_t* __restrict__ choice, float* __restrict__ route_w,
                                                        const float* __restrict__ ss, int ss_stride, int ss_count, float d, float eps,
                                                        float* __restrict__ row_rs) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= *m_count) return;
  float sq = 0.f;   // the row's sum of squares, for the expert GEMM
  if (row_rs)
    for (int i = lane; i < ss_count; i += 64) sq += ss[(size_t)row * ss_stride + i];
  float v[4];
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = lane + 64 * j;
    v[j] = e < E ? logits[(size_t)row * E + e] + 0.0f : -INFINITY;   // (-0 becomes +0: the two are a tie)
    m = fmaxf(m, v[j]);
  }
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  // top-k of the logits (softmax is monotone), lowest index on ties: the order of the logits as unsigned numbers, its maximum
  // by DPP moves inside the rows of 16 lanes and four scalar reads, and the first lane that holds it from a ballot (a maximum
  // over 64-bit (value, index) keys by six exchanges through LDS: 5.5 us per launch of 144 rows for 4.6 now).
  uint32_t ord[4];   // 0: not a choice
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t b = __float_as_uint(v[j]);
    ord[j] = v[j] > -INFINITY ? (b & 0x80000000u ? ~b : b | 0x80000000u) : 0u;
  }
  float wsel = 0.f;      // lane k keeps the k-th selected probability (the common factor 1/Z cancels in the renormalisation)
  int esel = -1;
  float wsum = 0.f;
  for (int k = 0; k < top_k; ++k) {
    uint32_t o = max(max(ord[0], ord[1]), max(ord[2], ord[3]));
    o = max(o, (uint32_t)__builtin_amdgcn_mov_dpp((int)o, 0xb1, 0xf, 0xf, true));    // lane ^ 1
    o = max(o, (uint32_t)__builtin_amdgcn_mov_dpp((int)o, 0x4e, 0xf, 0xf, true));    // lane ^ 2
    o = max(o, (uint32_t)__builtin_amdgcn_mov_dpp((int)o, 0x141, 0xf, 0xf, true));   // the other four of the half row
    o = max(o, (uint32_t)__builtin_amdgcn_mov_dpp((int)o, 0x140, 0xf, 0xf, true));   // the other half of the row
    const uint32_t best = max(max((uint32_t)__builtin_amdgcn_readlane((int)o, 0), (uint32_t)__builtin_amdgcn_readlane((int)o, 16)),
                              max((uint32_t)__builtin_amdgcn_readlane((int)o, 32), (uint32_t)__builtin_amdgcn_readlane((int)o, 48)));
    int ce = 0;
#pragma unroll
    for (int j = 3; j >= 0; --j) {
      const unsigned long long at = __ballot(ord[j] == best);
      if (at) ce = 64 * j + __ffsll((long long)at) - 1;
    }
    const float bv = best & 0x80000000u ? __uint_as_float(best & 0x7fffffffu) : __uint_as_float(~best);
    const float pw = best ? __expf(bv - m) : 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (lane + 64 * j == ce) ord[j] = 0u;   // taken
    wsum += pw;
    if (lane == k) { wsel = pw; esel = ce; }
  }
  if (lane < top_k) {
    const int o = row * top_k + lane;
    choice[o] = esel;
    route_w[o] = wsel / wsum;
  }
  if (row_rs) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
    if (lane == 0) row_rs[row] = 1.0f / sqrtf(sq / d + eps);
  }
}

// One workgroup: group offsets, the list of row tiles, the expert-sorted slot list; re-arms the counters.
// A thread keeps its slots' choices in registers between the two passes and requests them eight at a time (read one
// per loop iteration, 16 K slots cost 32 dependent L2 round trips per thread); the tile list is written by one thread
// per expert after a scan that touches LDS only.
__global__ __launch_bounds__(1024) void moe_group_kernel(int E, int top_k, const int32_t* __restrict__ m_count,
                                                         const int32_t* __restrict__ choice,
                                                         int32_t* __restrict__ sorted, int32_t* __restrict__ tile_expert,
                                                         int32_t* __restrict__ tile_row0, int32_t* __restrict__ tile_rows,
                                                         int32_t* __restrict__ n_tiles, int tile_cap, int lists) {
  __shared__ int s_class[64], s_nt[MOE_MAX_E + 8];
  __shared__ int s_off[MOE_MAX_E], s_tile0[MOE_MAX_E];
  __shared__ int s_cnt[MOE_MAX_E], s_fill[MOE_MAX_E];
  const int tid = threadIdx.x;
  const int total = *m_count * top_k;
  constexpr int KEEP = 24;   // slots per thread held in registers (24 K slots); the rest is read again in the second pass
  int mine[KEEP];
#pragma unroll
  for (int j0 = 0; j0 < KEEP; j0 += 8) {
#pragma unroll
    for (int j = j0; j < j0 + 8; ++j) mine[j] = (tid + j * 1024 < total) ? choice[tid + j * 1024] : -1;
  }
  for (int e = tid; e < E; e += 1024) { s_cnt[e] = 0; s_fill[e] = 0; }
  if (tid < 64) s_class[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < KEEP; ++j)
    if (mine[j] >= 0) atomicAdd(&s_cnt[mine[j]], 1);
  for (int i = tid + KEEP * 1024; i < total; i += 1024) atomicAdd(&s_cnt[choice[i]], 1);
  __syncthreads();
  if (tid < 64) {   // offsets of the groups and of their tiles: a scan by one wavefront, four experts per lane
    int c[4], run = 0, t = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      c[j] = 4 * tid + j < E ? s_cnt[4 * tid + j] : 0;
      run += c[j];
      t += (c[j] + 127) >> 7;
    }
    int ri = run, ti = t;   // inclusive over the lanes
    for (int off = 1; off < 64; off <<= 1) {
      const int a = __shfl_up(ri, off, 64), b = __shfl_up(ti, off, 64);
      if (tid >= off) { ri += a; ti += b; }
    }
    run = ri - run;
    t = ti - t;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (4 * tid + j < E) {
        s_off[4 * tid + j] = run;
        s_tile0[4 * tid + j] = t;
        run += c[j];
        t += (c[j] + 127) >> 7;
      }
    if (tid == 63 && lists == 0) *n_tiles = min(ti, tile_cap);
  }
  __syncthreads();
  if (lists > 0) {
    // Experts by falling row count (in classes of 16 rows; in which order within one does not matter) to the lists 0 .. L - 1, L - 1 .. 0, 0 .. L - 1: about as
    // many rows each, an expert's tiles next to each other on one of them.  Tiles of up to 256 rows, an expert's all alike.
    // Experts without a row come last, in a class of their own: dealt out among those of up to 15 rows they leave one XCD with five experts where
    // another has one, and a launch takes as long as the fullest.  9 rows (19 to 26 of 64 experts), us a launch, among / behind them: gate / up
    // 54.8 / 37.7, down 28.9 / 21.5.
    const int c = tid < E ? s_cnt[tid] : 0, cls = c > 0 ? 62 - min(62, c >> 4) : 63;
    int nt = (c + 255) >> 8;
    const int per = nt > 0 ? ((c + nt - 1) / nt + 15) & ~15 : 16;
    nt = (c + per - 1) / per;
    if (tid < E) atomicAdd(&s_class[cls], 1);
    __syncthreads();
    if (tid < 64) {   // experts in the classes ahead
      const int k = s_class[tid];
      int at = k;
      for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(at, off, 64);
        if (tid >= off) at += o;
      }
      s_class[tid] = at - k;
    }
    __syncthreads();
    const int rank = tid < E ? atomicAdd(&s_class[cls], 1) : 0, last = lists - 1, turn = rank / lists;   // (lists: a power of two)
    const int list = turn & 1 ? last - (rank & last) : rank & last;
    if (tid < E) s_nt[rank] = nt;
    __syncthreads();
    if (tid < E) {
      int t = list * tile_cap;
      for (int k = 0; k < turn; ++k) t += s_nt[lists * k + (k & 1 ? last - list : list)];
      for (int i = 0; i < nt && t < (list + 1) * tile_cap; ++i, ++t) {
        tile_expert[t] = tid;
        tile_row0[t] = s_off[tid] + i * per;
        tile_rows[t] = min(per, c - i * per);
      }
    }
    if (tid < 8) {
      int t = 0;
      for (int k = 0; tid < lists && lists * k < E; ++k) {
        const int r = lists * k + (k & 1 ? last - tid : tid);
        t += r < E ? s_nt[r] : 0;
      }
      n_tiles[tid] = min(t, tile_cap);   // (lists that there are not: none)
    }
  } else {
    for (int e = tid; e < E; e += 1024) {
      const int c = s_cnt[e], run = s_off[e];
      int t = s_tile0[e];
      for (int r0 = 0; r0 < c && t < tile_cap; r0 += 128, ++t) {
        tile_expert[t] = e;
        tile_row0[t] = run + r0;
        tile_rows[t] = min(128, c - r0);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < KEEP; ++j)
    if (mine[j] >= 0) sorted[s_off[mine[j]] + atomicAdd(&s_fill[mine[j]], 1)] = tid + j * 1024;
  for (int i = tid + KEEP * 1024; i < total; i += 1024) {
    const int e = choice[i];
    sorted[s_off[e] + atomicAdd(&s_fill[e], 1)] = i;
  }
}

// h[row] += sum over slots (in slot order) of y[row, slot]; also the operand and the partial sums
// of squares of the next norm (one number per row).
__global__ __launch_bounds__(256) void moe_combine_kernel(const float* __restrict__ y, int d, int top_k,
                                                          const int32_t* __restrict__ m_count, float* __restrict__ h,
                                                          bf16_t* __restrict__ xg, int xg_ld, int xg_lo,
                                                          const float* __restrict__ gain_next,
                                                          float* __restrict__ ss, int ss_stride) {
  const int row = blockIdx.x;
  if (row >= *m_count) return;
  __shared__ float s_sq[4];
  float sq = 0.f;
  constexpr int SLOTS = 8;   // requested at once (one by one: 8.0 us per launch of 144 rows and eight slots for 6.1)
  for (int c = threadIdx.x * 4; c < d; c += 1024) {
    float4 acc = *(const float4*)(h + (size_t)row * d + c);
    for (int k0 = 0; k0 < top_k; k0 += SLOTS) {
      float4 t[SLOTS];
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) t[k] = *(const float4*)(y + ((size_t)row * top_k + min(k0 + k, top_k - 1)) * d + c);
#pragma unroll
      for (int k = 0; k < SLOTS; ++k)
        if (k0 + k < top_k) { acc.x += t[k].x; acc.y += t[k].y; acc.z += t[k].z; acc.w += t[k].w; }
    }
    *(float4*)(h + (size_t)row * d + c) = acc;
    const float4 gn = *(const float4*)(gain_next + c);
    const float xv[4] = {acc.x * gn.x, acc.y * gn.y, acc.z * gn.z, acc.w * gn.w};
    act_put4(xg, xg_lo, row, c, xg_ld, xv[0], xv[1], xv[2], xv[3]);
    sq += (acc.x * acc.x + acc.y * acc.y) + (acc.z * acc.z + acc.w * acc.w);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
  if ((threadIdx.x & 63) == 0) s_sq[threadIdx.x >> 6] = sq;
  __syncthreads();
  if (threadIdx.x == 0) ss[(size_t)row * ss_stride] = (s_sq[0] + s_sq[1]) + (s_sq[2] + s_sq[3]);
}

__global__ void moe_copy_choices_kernel(const int32_t* __restrict__ src, int32_t* __restrict__ dst, int layers,
                                        int per_layer_src, int per_layer_dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= layers * per_layer_dst) return;
  dst[i] = src[(size_t)(i / per_layer_dst) * per_layer_src + i % per_layer_dst];
}

void launch_moe_route(hipStream_t st, const float* logits, int E, int top_k, const int32_t* m_count, int rows_cap,
                      int32_t* choice, float* route_w, const float* ss, int ss_stride, int ss_count, int d, float eps,
                      float* row_rs) {
  S2D2_LAUNCH(moe_route_kernel, dim3((rows_cap + 3) / 4), dim3(256), 0, st, logits, E, top_k, m_count, choice,
                     route_w, ss, ss_stride, ss_count, (float)d, eps, row_rs);
}

void launch_moe_group(hipStream_t st, int E, int top_k, const int32_t* m_count, const int32_t* choice,
                      int32_t* sorted, int32_t* tile_expert, int32_t* tile_row0, int32_t* tile_rows, int32_t* n_tiles,
                      int tile_cap, int lists) {
  S2D2_LAUNCH(moe_group_kernel, dim3(1), dim3(1024), 0, st, E, top_k, m_count, choice, sorted,
                     tile_expert, tile_row0, tile_rows, n_tiles, tile_cap, lists);
}

void launch_moe_combine(hipStream_t st, const float* y, int d, int top_k, const int32_t* m_count, int rows_cap,
                        float* h, void* xg, int xg_ld, int xg_lo, const float* gain_next, float* ss, int ss_stride) {
  S2D2_LAUNCH(moe_combine_kernel, dim3(rows_cap), dim3(256), 0, st, y, d, top_k, m_count, h, (bf16_t*)xg,
                     xg_ld, xg_lo, gain_next, ss, ss_stride);
}

void launch_moe_copy_choices(hipStream_t st, const int32_t* src, int32_t* dst, int layers, int per_layer_src,
                             int per_layer_dst) {
  const int n = layers * per_layer_dst;
  S2D2_LAUNCH(moe_copy_choices_kernel, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, layers, per_layer_src,
                     per_layer_dst);
}

}  // namespace s2d2
