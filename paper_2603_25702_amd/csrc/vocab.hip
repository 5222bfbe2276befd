// Vocabulary-wide kernels: SampleFromLogits / ScoreFromLogits statistics, the threshold set of
// Algorithm 2, and the accept scan + residual resampling of Algorithm 3.
//
// The statistics kernels stream each fp32 logit row exactly once with 16-byte coalesced loads
// (HBM-bound: rows * V * 4 bytes), keep an online (max, sum-exp, entropy numerator, arg-max,
// second max) per lane, and reduce with wavefront shuffles, then LDS, then a fixed-order merge
// over the row's chunks, so results do not depend on scheduling.
#include "s2d2_internal.h"
#include "../../include/s2d2.h"

#include <mutex>
#include <type_traits>

namespace s2d2 {

// Logits per workgroup: 256 lanes x VT float4, all in flight at once.  Eight float4 per lane take longer at every size, us per
// launch, four / eight: rows of 151936 logits (38 workgroups each) 4 rows 4.9 / 7.1, 64 11.3 / 11.8, 256 28.2 / 32.5, 1024 98 / 106;
// rows of 40000 (10 each) 64 rows 6.0 / 8.1, 1024 29.3 / 34.6.
static constexpr int VT = 4;

// Workgroups that share the draw of a row: as many as there are compute units for (256; the workspace is sized without a device to ask),
// at most eight.  One / two / four / eight / sixteen, us per launch, rows of 151936 logits: 4 rows 32.4 / 21.9 / 16.4 / 11.7 / 11.2, 16
// 33.0 / 22.0 / 16.7 / 12.5 / 13.6, 64 39.1 / 26.6 / 20.2 / 22.8 / 36.7, 128 41.1 / 29.5 / 36.2, 256 44.5 / 53.6.
static int sample_share(int rows) { return std::max(1, std::min(8, 256 / rows)); }
int sample_rows_shared(int rows) { return std::min(rows, 128); }   // most rows with more than one

// Workgroups of the statistics, and most chunks that one walks.  1024 / 4096 / 8192 / 16384 workgroups / one a
// chunk, us, rows of 151936 logits: 4 rows 5.6 in all, 64 12.2 / 10.8 / 10.8 / 10.8 / 10.9, 256 31.5 / 28.5 / 28.7 / 30.3 / 30.8, 512 55.8 / 54.4 / 52.4 / 52.5 /
// 58.9, 1024 (runs of 38, 10, 5, 3 and 1 chunks) 103.3 / 105.8 / 102.3 / 99.2 / 112.1.  Behind a forward, that is with the logits' last quarter in the memory-side
// cache, runs of 5 / 3 / 2 / 1 chunks, in brackets a workgroup per chunk and a launch for the merge: 1024 rows of the MoE shape 115 / 112 / 113 / 116 (113), of the 1.7B
// one 112 / 109 / 108 / 115 (109), 4B verification 109 / 104 / 104 / 111 (111); 768 rows of 8B, 4 / 3 / 2 / 1 84 / 80 / 81 / 88 (88), 512, 3 / 2 / 1 54 / 57 / 62 (60).
static constexpr int STATS_WGS = 8192, STATS_MOST = 3;

int vocab_chunks(int V) { return (V + 1024 * VT - 1) / (1024 * VT); }

struct Stat {
  float m;    // max logit
  float z;    // sum exp(l - m)
  float e;    // sum exp(l - m) * (l - m)
  float m2;   // second largest logit (equals m if the max is attained twice)
  int arg;    // lowest index attaining m
};

__device__ __forceinline__ Stat stat_empty() { return Stat{-INFINITY, 0.f, 0.f, -INFINITY, 0x7fffffff}; }

__device__ __forceinline__ Stat stat_merge(const Stat& a, const Stat& b) {
  Stat r;
  r.m = fmaxf(a.m, b.m);
  r.arg = a.m > b.m ? a.arg : (b.m > a.m ? b.arg : min(a.arg, b.arg));
  r.m2 = fmaxf(fminf(a.m, b.m), fmaxf(a.m2, b.m2));
  const float da = a.m - r.m, db = b.m - r.m;  // <= 0, or NaN when both are -inf
  const float fa = a.z > 0.f ? __expf(da) : 0.f, fb = b.z > 0.f ? __expf(db) : 0.f;
  r.z = a.z * fa + b.z * fb;
  r.e = (a.z > 0.f ? fa * (a.e + da * a.z) : 0.f) + (b.z > 0.f ? fb * (b.e + db * b.z) : 0.f);
  return r;
}

__device__ __forceinline__ Stat stat_shfl_xor(const Stat& s, int off) {
  Stat r;
  r.m = __shfl_xor(s.m, off, 64);
  r.z = __shfl_xor(s.z, off, 64);
  r.e = __shfl_xor(s.e, off, 64);
  r.m2 = __shfl_xor(s.m2, off, 64);
  r.arg = __shfl_xor(s.arg, off, 64);
  return r;
}

// Reductions over a wavefront in a fixed order, the same result in every lane: a butterfly of DPP moves inside the rows of 16
// lanes (vector-ALU operands, no LDS trip), two exchanges between the rows.
template <typename F>
__device__ __forceinline__ float wave_all(float v, const F& op) {
  auto row = [&](auto ctrl) __attribute__((always_inline)) {
    v = op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true)));
  };
  row(std::integral_constant<int, 0xb1>{});    // lane ^ 1
  row(std::integral_constant<int, 0x4e>{});    // lane ^ 2
  row(std::integral_constant<int, 0x141>{});   // the other four of the half row
  row(std::integral_constant<int, 0x140>{});   // the other half of the row
  v = op(v, __shfl_xor(v, 16, 64));
  return op(v, __shfl_xor(v, 32, 64));
}

// What becomes of a row's statistics: outputs at [sequence of the row][block index], or [row] without logit_seq.
struct VocabOut {
  const int32_t *logit_seq, *logit_idx;
  int B;
  const int32_t* token;                      // scores: the token of each place
  int32_t* xhat;                             // proposals and their statistics
  float *p, *lse, *margin, *entropy_n, *q;   // (q and lse: scores)
};
__device__ __forceinline__ int vocab_place(const VocabOut& f, int row) { return f.logit_seq ? f.logit_seq[row] * f.B + f.logit_idx[row] : row; }

// SampleFromLogits (greedy): x_hat = arg-max, p = softmax probability of it, plus lse, margin, H/ln V.
// ScoreFromLogits: q = softmax(logits_ver)[token], lse.  tok, x: the token and its logit.
template <bool SCORE>
__device__ __forceinline__ void vocab_finish(const Stat& s, const VocabOut& f, int o, int V, int tok, float x) {
  const float l = s.m + logf(s.z);
  f.lse[o] = l;
  if (SCORE) {
    f.q[o] = (tok >= 0 && tok < V) ? expf(x - l) : 0.f;
  } else {
    const float inv = 1.0f / s.z;
    f.xhat[o] = s.arg < V ? s.arg : 0;   // no comparable logit in the row (all NaN): the first index, as an arg-max over NaNs gives
    f.p[o] = inv;
    f.margin[o] = inv - expf(s.m2 - s.m) * inv;
    f.entropy_n[o] = fmaxf(0.f, logf(s.z) - s.e * inv) / logf((float)V);
  }
}

// part[row][chunk][8] = {m, z, e, m2, arg}; the workgroup of a row that counts its arrival last merges the row's chunks and finishes it
// (arrive: a counter per row, zero between launches): a lane per chunk, then a butterfly over the lanes, a fixed order (stat_merge is
// symmetric, ties go to the lower index).  Nobody waits for another workgroup.
// inv_t: 1 / temperature (1 in greedy mode: the multiplication is then exact); all statistics are those of
// softmax(logits * inv_t).
//
// Bound: reading the logits, with the vector ALU close behind (ten instructions and an exponential a logit).  The exponentials
// are taken against the wavefront's maximum, so that only sums are left to reduce over its lanes; with each lane's own maximum
// and a merge of whole statistics (five exchanges, two exponentials, six times over) the merge was half of the instructions.
// A workgroup walks a run of chunks with the next one requested and arrives once.  Rows of 151936 logits, us, a workgroup per chunk and a launch
// behind it for the merge / now: 4 rows 4.9 + 4.5 / 5.6, 64 14.9 / 10.8, 128 20.4 / 16.4, 256 32.1 / 28.7 (5.4 TB/s), 512 55.9 / 52.4, 1024 103.9 / 99.2 (6.3 TB/s)
// (with the arrival counters of all rows in one stretch of memory and an arrival per chunk: 256 rows 50).
template <bool SCORE>
__global__ __launch_bounds__(256) void vocab_stats_kernel(const float* __restrict__ logits, int V, const int32_t* __restrict__ count,
                                                          int chunks, int per, float inv_t, float* __restrict__ part, int32_t* __restrict__ arrive,
                                                          const VocabOut f) {
  __shared__ Stat s_w[STATS_MOST][4];
  const int row = blockIdx.y, c0 = blockIdx.x * per, mine = min(per, chunks - c0);   // chunks c0 .. c0 + mine - 1
  if (count && row >= *count) return;
  const float* x = logits + (size_t)row * V;
  const int tid = threadIdx.x;
  auto load = [&](int c, f32x4_t (&v)[VT], auto vec) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < VT; ++t) {
      const int i = (c0 + c) * 1024 * VT + t * 1024 + tid * 4;
      if (decltype(vec)::value) v[t] = ld_stream((const f32x4_t*)(x + min(i, V - 4)));   // (past the end: not looked at)
      else
#pragma unroll
        for (int e = 0; e < 4; ++e) v[t][e] = x[min(i + e, V - 1)];
    }
  };
  // statistics of one chunk's logits, over the wavefront
  auto reduce = [&](int c, const f32x4_t (&r)[VT]) __attribute__((always_inline)) {
    const int base = (c0 + c) * 1024 * VT;
    float v[4 * VT];
#pragma unroll
    for (int t = 0; t < 4 * VT; ++t) v[t] = r[t >> 2][t & 3] * inv_t;
    if (base + 1024 * VT > V) {   // (the last chunk of a row)
#pragma unroll
      for (int t = 0; t < 4 * VT; ++t) v[t] = base + (t >> 2) * 1024 + tid * 4 + (t & 3) < V ? v[t] : -INFINITY;
    }
    float lm = -INFINITY, lm2 = -INFINITY;   // this lane's largest and second largest logit; the place of the first largest
    int at = 0;
#pragma unroll
    for (int t = 0; t < 4 * VT; ++t) {
      at = v[t] > lm ? t : at;
      lm2 = __builtin_amdgcn_fmed3f(v[t], lm, lm2);
      lm = fmaxf(lm, v[t]);
    }
    auto larger = [](float a, float b) __attribute__((always_inline)) { return fmaxf(a, b); };
    auto sum = [](float a, float b) __attribute__((always_inline)) { return a + b; };
    Stat s = stat_empty();
    s.m = wave_all(lm, larger);
    const bool own = lm > -INFINITY;   // (a lane without a comparable logit adds nothing)
    float z = 0.f, e = 0.f;
    if (own) {
#pragma unroll
      for (int t = 0; t < 4 * VT; ++t) {
        const float d = v[t] - s.m;
        const float ex = __expf(d);          // exp(-inf) = 0 for padded slots
        z += ex;
        e = __builtin_fmaf(ex, fmaxf(d, -200.f), e);   // (-inf would make 0 * -inf; exp is 0 well above -200)
      }
    }
    s.z = wave_all(z, sum);
    s.e = wave_all(e, sum);
    const unsigned long long top = __ballot(own && lm == s.m);   // the lanes that hold the maximum
    const bool one = __popcll(top) == 1;
    s.m2 = wave_all(one && lm == s.m ? lm2 : lm, larger);
    if (top) {
      const int i = base + (at >> 2) * 1024 + tid * 4 + (at & 3);
      s.arg = __builtin_amdgcn_readlane(i, __ffsll((long long)top) - 1);
      if (!one)
        for (unsigned long long rest = top & (top - 1); rest; rest &= rest - 1) s.arg = min(s.arg, __builtin_amdgcn_readlane(i, __ffsll((long long)rest) - 1));
    }
    if ((tid & 63) == 0) s_w[c][tid >> 6] = s;
  };
  auto walk = [&](auto vec) __attribute__((always_inline)) {   // a chunk is requested ahead of the one before it being reduced
    f32x4_t a[VT], b[VT];
    load(0, a, vec);
    for (int c = 0; c < mine; c += 2) {
      if (c + 1 < mine) load(c + 1, b, vec);
      reduce(c, a);
      if (c + 1 < mine) {
        if (c + 2 < mine) load(c + 2, a, vec);
        reduce(c + 1, b);
      }
    }
  };
  if ((V & 3) == 0) walk(std::true_type{});
  else walk(std::false_type{});
  const int o = vocab_place(f, row);
  int tok = 0;
  float xt = 0.f;
  if (SCORE) {
    tok = f.token[o];
    xt = x[tok >= 0 && tok < V ? tok : 0] * inv_t;
  }
  __syncthreads();
  if (tid >= 64) return;
  Stat r = stat_empty();
  if (tid < mine) r = stat_merge(stat_merge(s_w[tid][0], s_w[tid][1]), stat_merge(s_w[tid][2], s_w[tid][3]));
  if (gridDim.x > 1) {
    if (tid < mine) {
      float* po = part + ((size_t)row * chunks + c0 + tid) * 8;
      st16f_coh(po, r.m, r.z, r.e, r.m2);
      st4f_coh(po + 4, __int_as_float(r.arg));
    }
    __builtin_amdgcn_s_waitcnt(0);   // the write-through stores have completed before the arrival is counted
    int last = 0;
    if (tid == 0) {
      last = __hip_atomic_fetch_add(&arrive[row * ARRIVE_STRIDE], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
      if (last) __hip_atomic_store(&arrive[row * ARRIVE_STRIDE], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    r = stat_empty();
    for (int c = tid; c < chunks; c += 64) {
      const float* pc = part + ((size_t)row * chunks + c) * 8;
      r = stat_merge(r, Stat{ld4f_coh(pc), ld4f_coh(pc + 1), ld4f_coh(pc + 2), ld4f_coh(pc + 3), __float_as_int(ld4f_coh(pc + 4))});
    }
  }
  for (int off = 1; off < 64; off <<= 1) r = stat_merge(r, stat_shfl_xor(r, off));
  if (tid == 0) vocab_finish<SCORE>(r, f, o, V, tok, xt);
}

template <bool SCORE>
static void launch_stats(hipStream_t st, const float* logits, int V, const int32_t* count, int rows_cap, const VocabWs& ws, float inv_t, const VocabOut& f) {
  const int wgs = std::max(1, STATS_WGS / rows_cap), per = std::min((ws.chunks + wgs - 1) / wgs, STATS_MOST);
  S2D2_LAUNCH((vocab_stats_kernel<SCORE>), dim3((ws.chunks + per - 1) / per, rows_cap), dim3(256), 0, st, logits, V, count, ws.chunks, per, inv_t, ws.part,
              ws.arrive, f);
}

__global__ void vocab_sample_kernel(const float* __restrict__ logits, int V, const int32_t* __restrict__ count,
                                    const int32_t* __restrict__ logit_seq, const int32_t* __restrict__ logit_idx, int B,
                                    uint64_t seed, uint32_t step, const uint32_t* __restrict__ step_dev, float inv_t,
                                    const float* __restrict__ lse, int32_t* __restrict__ xhat, float* __restrict__ p,
                                    float* __restrict__ tile_scratch, int32_t* __restrict__ arrivals);

void launch_vocab_draft(hipStream_t st, const float* logits, int V, const int32_t* count, int rows_cap,
                        const VocabWs& ws, const int32_t* logit_seq, const int32_t* logit_idx, int B,
                        int32_t* xhat, float* p, float* lse, float* margin, float* entropy_n, const VocabSample& sm) {
  const float inv_t = sm.sample ? 1.0f / sm.temperature : 1.0f;
  launch_stats<false>(st, logits, V, count, rows_cap, ws, inv_t, VocabOut{logit_seq, logit_idx, B, nullptr, xhat, p, lse, margin, entropy_n, nullptr});
  if (sm.sample)
    S2D2_LAUNCH(vocab_sample_kernel, dim3(rows_cap, sample_share(rows_cap)), dim3(1024), 0, st, logits, V, count, logit_seq, logit_idx, B,
                sm.seed, sm.step, sm.step_dev, inv_t, lse, xhat, p, ws.sample_tiles, ws.sample_arrive);
}

void launch_vocab_score(hipStream_t st, const float* logits, int V, const int32_t* count, int rows_cap,
                        const VocabWs& ws, const int32_t* logit_seq, const int32_t* logit_idx, int B,
                        const int32_t* token, float* q, float* lse, float inv_t) {
  launch_stats<true>(st, logits, V, count, rows_cap, ws, inv_t, VocabOut{logit_seq, logit_idx, B, token, nullptr, nullptr, lse, nullptr, nullptr, q});
}

// Per sequence: defaults for committed positions, threshold set S = {i in M: p_i > tau} U {argmax p}.
__global__ void draft_finish_kernel(int N, int B, int mask_id, float tau, const int32_t* __restrict__ block,
                                    int32_t* __restrict__ xhat, float* __restrict__ p, float* __restrict__ lse,
                                    float* __restrict__ margin, float* __restrict__ entropy_n,
                                    uint64_t* __restrict__ unmask, int32_t* __restrict__ n_hi) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  uint64_t bits = 0;
  int hi = 0, best = -1;
  float best_p = -1.f;
  for (int i = 0; i < B; ++i) {
    const int o = n * B + i;
    if (block[o] == mask_id) {
      const float pi = p[o];
      if (pi > tau) { bits |= 1ull << i; ++hi; }
      if (pi > best_p) { best_p = pi; best = i; }   // strict: lowest index wins ties
    } else {
      xhat[o] = -1; p[o] = 0.f; lse[o] = 0.f; margin[o] = 0.f; entropy_n[o] = 0.f;
    }
  }
  if (best >= 0) bits |= 1ull << best;
  unmask[n] = bits;
  n_hi[n] = hi;
}

void launch_draft_finish(hipStream_t st, int N, int B, int mask_id, float tau, const int32_t* block,
                         int32_t* xhat, float* p, float* lse, float* margin, float* entropy_n,
                         uint64_t* unmask, int32_t* n_hi) {
  S2D2_LAUNCH(draft_finish_kernel, dim3((N + 63) / 64), dim3(64), 0, st, N, B, mask_id, tau, block, xhat, p,
                     lse, margin, entropy_n, unmask, n_hi);
}

// ---------------------------------------------------------------------------------------------
// Counter-based uniforms: Philox-4x32 with 10 rounds (Salmon et al., SC'11), written from the
// published round function.  key = seed, counter = (step, sequence, block index, stream).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t philox_first_word(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                      uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    c0 = hi1 ^ c1 ^ k0;
    c1 = lo1;
    c2 = hi0 ^ c3 ^ k1;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}

__device__ __forceinline__ float uniform01(uint64_t seed, uint32_t step, uint32_t seq, uint32_t idx, uint32_t stream) {
  const uint32_t w = philox_first_word(step, seq, idx, stream, (uint32_t)seed, (uint32_t)(seed >> 32));
  return ((float)(w >> 9) + 0.5f) * (1.0f / 8388608.0f);  // odd multiple of 2^-24: exact
}

// Scan of one non-negative float per thread over a 256-thread block with a fixed tree.
// Returns the inclusive prefix; *excl is the inclusive prefix of the previous thread (0 for
// thread 0), so the intervals [excl, incl) of consecutive threads tile [0, total) exactly;
// *total is the inclusive prefix of the last thread.  s_w needs 4 floats.  Threads past the first 256 (a wider
// workgroup) must pass 0 and get an empty interval at the total.
__device__ __forceinline__ float block_scan_256(float v, float* s_w, float* excl, float* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int off = 1; off < 64; off <<= 1) {
    const float t = __shfl_up(v, off, 64);
    if (lane >= off) v += t;
  }
  __syncthreads();
  if (lane == 63 && w < 4) s_w[w] = v;
  __syncthreads();
  float pre = 0.f;
  for (int i = 0; i < min(w, 4); ++i) pre += s_w[i];
  const float incl = v + pre;
  const float prev = __shfl_up(incl, 1, 64);
  *excl = lane == 0 ? pre : prev;
  *total = s_w[3] + ((s_w[0] + s_w[1]) + s_w[2]);
  return incl;
}

static constexpr int RTILE = 256;     // residual tile: one wavefront x float4
static constexpr int RMAX_TILES = 8192;

// Inverse CDF over V non-negative weights in ascending index order, by a workgroup of 256 threads or more (the tile sums use all of them):
// returns (in the lanes of wavefront 0; -1 elsewhere) the smallest index whose inclusive prefix sum exceeds
// u * total, or -1 if the weights have no mass.  w4(i0, r) yields the weights of indices i0 .. i0+3 (zeros
// past V).  Two levels with a fixed summation order: tile sums (256 indices per tile: one wavefront x 4),
// a scan of the tile sums, then a walk of the selected tile; rounding at either level falls back to the
// nearest index that has mass.  s_tile needs RMAX_TILES floats, s_w four.
// First level: the sums of tiles [tb, te) go to dst[tile] (LDS, or global memory with device-coherent stores when
// several workgroups share the tiles of one row).  Eight tiles of a wavefront at a time: their loads are all issued
// before the first reduction (one tile per iteration made the pass a chain of ~150 memory round trips per
// wavefront).  A tile's sum does not depend on which wavefront or workgroup forms it.
template <bool COH, typename F>
__device__ __forceinline__ void inverse_cdf_tile_sums(const F& w4, int tb, int te, float* dst) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int TU = 8;
  const int nw = blockDim.x >> 6;   // every wavefront of the workgroup takes part in this pass; the scan uses 256 threads
  for (int t0 = tb + w * TU; t0 < te; t0 += nw * TU) {
    float r4[TU][4];
#pragma unroll
    for (int u_ = 0; u_ < TU; ++u_) w4((t0 + u_) * RTILE + lane * 4, r4[u_]);   // indices at or past V give zeros
#pragma unroll
    for (int u_ = 0; u_ < TU; ++u_) {
      float r = ((r4[u_][0] + r4[u_][1]) + r4[u_][2]) + r4[u_][3];
      for (int off = 32; off > 0; off >>= 1) r += __shfl_xor(r, off, 64);
      if (lane == 0 && t0 + u_ < te) {
        if (COH) st4f_coh(&dst[t0 + u_], r); else dst[t0 + u_] = r;
      }
    }
  }
}

// Second and third level, from the tile sums in s_tile (written by this workgroup's threads before the call).
template <typename F>
__device__ __forceinline__ int inverse_cdf_finish(const F& w4, int V, float u, float* s_tile, float* s_w,
                                                  int* s_tile_sel, float* s_before) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int tiles = (V + RTILE - 1) / RTILE;
  __syncthreads();
  // scan tile sums: thread t owns tiles [t*per, (t+1)*per)
  const int per = (tiles + 255) / 256;   // (threads past the first 256 own no tiles)
  float mine = 0.f;
  for (int t = tid * per; t < min(tiles, (tid + 1) * per); ++t) mine += s_tile[t];
  float total, excl;
  const float incl = block_scan_256(mine, s_w, &excl, &total);
  const float target = u * total;
  if (tid == 0) { *s_tile_sel = -1; *s_before = 0.f; }
  __syncthreads();
  if (excl <= target && target < incl) {  // exactly one thread: the intervals tile [0, total)
    float run = excl, before = excl;
    int sel = -1, last = -1;
    for (int t = tid * per; t < min(tiles, (tid + 1) * per); ++t) {
      const float ts = s_tile[t];
      if (ts > 0.f) { last = t; before = run; }
      if (ts > 0.f && run + ts > target) { sel = t; break; }
      run += ts;
    }
    if (sel < 0) sel = last;          // rounding: take the thread's last tile that has mass
    *s_tile_sel = sel;
    *s_before = before;
  }
  __syncthreads();
  int sel = *s_tile_sel;
  int token = -1;
  if (total > 0.f && sel < 0) {  // target landed at or beyond the total by rounding: last tile with mass
    if (tid == 0) {
      for (int t = tiles - 1; t >= 0; --t)
        if (s_tile[t] > 0.f) { *s_tile_sel = t; break; }
      float run = 0.f;
      for (int t = 0; t < *s_tile_sel; ++t) run += s_tile[t];
      *s_before = run;
    }
    __syncthreads();
    sel = *s_tile_sel;
  }
  if (total > 0.f && sel >= 0 && w == 0) {  // wave 0 walks the selected tile in index order
    const int i0 = sel * RTILE + lane * 4;
    float r4[4];
    w4(i0, r4);
    const float ls = ((r4[0] + r4[1]) + r4[2]) + r4[3];
    float inc = ls;
    for (int off = 1; off < 64; off <<= 1) {
      const float t = __shfl_up(inc, off, 64);
      if (lane >= off) inc += t;
    }
    float run = *s_before + (inc - ls);
    int cand = 0x7fffffff, last_pos = -1;
    for (int e = 0; e < 4; ++e) {
      if (r4[e] > 0.f) last_pos = i0 + e;
      run += r4[e];
      if (cand == 0x7fffffff && r4[e] > 0.f && run > target) cand = i0 + e;
    }
    for (int off = 32; off > 0; off >>= 1) {
      cand = min(cand, __shfl_xor(cand, off, 64));
      last_pos = max(last_pos, __shfl_xor(last_pos, off, 64));
    }
    token = cand != 0x7fffffff ? cand : last_pos;
  }
  return token;
}

template <typename F>
__device__ __forceinline__ int inverse_cdf_block(const F& w4, int V, float u, float* s_tile, float* s_w,
                                                 int* s_tile_sel, float* s_before) {
  inverse_cdf_tile_sums<false>(w4, 0, (V + RTILE - 1) / RTILE, s_tile);
  return inverse_cdf_finish(w4, V, u, s_tile, s_w, s_tile_sel, s_before);
}

// Tile sums of one row by the G workgroups that share it: each forms its share and leaves it in `sums` (device-coherent
// stores), counts its arrival, and the last one to arrive takes them all into s_tile and re-arms the counter.  False in the
// workgroups that are done.  Nobody waits for another workgroup.
template <typename F>
__device__ __forceinline__ bool share_tile_sums(const F& w4, int V, int g, int G, float* sums, int32_t* arrivals, float* s_tile, int* s_last) {
  const int tid = threadIdx.x, tiles = (V + RTILE - 1) / RTILE, share = (tiles + G - 1) / G;
  inverse_cdf_tile_sums<true>(w4, min(tiles, g * share), min(tiles, (g + 1) * share), sums);
  __builtin_amdgcn_s_waitcnt(0);   // the write-through stores have completed before the arrival is counted
  __syncthreads();
  if (tid == 0) {
    const int prev = __hip_atomic_fetch_add(arrivals, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_last = prev == G - 1;
    if (prev == G - 1) __hip_atomic_store(arrivals, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!*s_last) return false;
  for (int t = tid; t < tiles; t += blockDim.x) s_tile[t] = ld4f_coh(&sums[t]);
  return true;
}

// SampleFromLogits in sampling mode: x_hat ~ softmax(logits / T) by inverse CDF in ascending vocabulary order with
// the uniform of stream 2 at (step, sequence, block index); p = that token's probability.  gridDim.y workgroups per
// logit row; runs after the statistics kernels (reads lse, overwrites the arg-max proposal and its probability).
// Sixteen wavefronts: a row of 152k logits is one stream through one compute unit (with four, 105 us per launch at 64 rows).
// With few rows most compute units have none, so up to eight workgroups share a row (sample_share).  The sums
// of the tiles, and with them the result, do not depend on gridDim.y.
__global__ __launch_bounds__(1024) void vocab_sample_kernel(
    const float* __restrict__ logits, int V, const int32_t* __restrict__ count, const int32_t* __restrict__ logit_seq,
    const int32_t* __restrict__ logit_idx, int B, uint64_t seed, uint32_t step, const uint32_t* __restrict__ step_dev,
    float inv_t, const float* __restrict__ lse, int32_t* __restrict__ xhat, float* __restrict__ p, float* __restrict__ tile_scratch,
    int32_t* __restrict__ arrivals) {
  __shared__ float s_tile[RMAX_TILES];
  __shared__ float s_w[4];
  __shared__ int s_tile_sel, s_last;
  __shared__ float s_before;
  const int row = blockIdx.x;
  if (row >= *count) return;
  const int n = logit_seq ? logit_seq[row] : row, idx = logit_idx ? logit_idx[row] : 0;
  const int o = logit_seq ? n * B + idx : row;
  const float* x = logits + (size_t)row * V;
  const float z = lse[o];
  const uint32_t stp = step + (step_dev ? *step_dev : 0u);
  const float u = uniform01(seed, stp, (uint32_t)n, (uint32_t)idx, 2u);
  auto prob4 = [&](int i0, float (&r)[4]) {
    if ((V & 3) == 0) {   // unconditional load (clamped index) so that the loads of several tiles can be in flight
      const bool ok = i0 < V;
      const float4 a = *(const float4*)(x + (ok ? i0 : 0));
      r[0] = ok ? __expf(a.x * inv_t - z) : 0.f; r[1] = ok ? __expf(a.y * inv_t - z) : 0.f;
      r[2] = ok ? __expf(a.z * inv_t - z) : 0.f; r[3] = ok ? __expf(a.w * inv_t - z) : 0.f;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = (i0 + e < V) ? __expf(x[i0 + e] * inv_t - z) : 0.f;
    }
  };
  int token;
  if (gridDim.y == 1) {
    token = inverse_cdf_block(prob4, V, u, s_tile, s_w, &s_tile_sel, &s_before);
  } else {
    if (!share_tile_sums(prob4, V, blockIdx.y, gridDim.y, tile_scratch + (size_t)row * ((V + RTILE - 1) / RTILE), &arrivals[row * ARRIVE_STRIDE], s_tile, &s_last)) return;
    token = inverse_cdf_finish(prob4, V, u, s_tile, s_w, &s_tile_sel, &s_before);
  }
  if (threadIdx.x == 0 && token >= 0) {   // (no mass cannot happen for a softmax; the arg-max proposal would stay)
    xhat[o] = token;
    p[o] = expf(x[token] * inv_t - z);
  }
}

// gridDim.y workgroups per sequence: accept scan over C_t (thread 0 of each, the same result in all), then, if a
// drafted token failed, a draw from the residual (P_ver - P_draft)_+ by inverse CDF in ascending vocabulary order.
// With several workgroups each forms the tile sums of its share of the vocabulary (one sequence alone would stream
// its two logit rows through a single compute unit), leaves them in tile_scratch[sequence][tile] and counts its
// arrival; the last one to arrive finishes the draw and re-arms the counter.  Workgroup 0 writes everything that
// does not depend on the draw.  The result does not depend on gridDim.y.
__global__ __launch_bounds__(1024) void accept_kernel(
    int B, int V, uint64_t seed, uint32_t step, const uint32_t* __restrict__ step_dev, float gamma, int resample,
    float inv_t, const int32_t* __restrict__ span_start, const int32_t* __restrict__ span_len,
    const float* __restrict__ logits_d, const int32_t* __restrict__ row_of_d,
    const float* __restrict__ logits_v, const int32_t* __restrict__ row_of_v,
    const int32_t* __restrict__ xhat, const float* __restrict__ p, const float* __restrict__ lse_d,
    const float* __restrict__ q, const float* __restrict__ lse_v, int32_t* __restrict__ block,
    int32_t* __restrict__ n_accept, int32_t* __restrict__ n_commit, int32_t* __restrict__ resampled,
    float* __restrict__ u_used, const int32_t* __restrict__ active, float* __restrict__ tile_scratch,
    int32_t* __restrict__ arrivals) {
  __shared__ float s_tile[RMAX_TILES];
  __shared__ float s_w[4];
  __shared__ int s_nacc, s_last;
  __shared__ int s_tile_sel;
  __shared__ float s_before;
  const int n = blockIdx.x, tid = threadIdx.x, g = blockIdx.y, G = gridDim.y;
  const int j = span_start[n], L = (active && active[n] == 0) ? 0 : span_len[n];   // not routed to the verifier: nothing to scan
  const uint32_t stp = step + (step_dev ? *step_dev : 0u);
  if (g == 0)
    for (int i = tid; i < B; i += blockDim.x) u_used[(size_t)n * B + i] = 0.f;
  __syncthreads();
  if (tid == 0) {
    int acc = 0;
    for (; acc < L; ++acc) {
      const int o = n * B + j + acc;
      const float u = uniform01(seed, stp, (uint32_t)n, (uint32_t)(j + acc), 0u);
      if (g == 0) u_used[o] = u;
      const float pi = p[o], qi = q[o];
      const bool ok = gamma == 1.0f ? (u * pi < qi) : (u < fminf(1.0f, powf(qi / pi, gamma)));
      if (!ok) break;
    }
    s_nacc = acc;
  }
  __syncthreads();
  const int acc = s_nacc;
  if (g == 0)
    for (int i = tid; i < acc; i += blockDim.x) block[n * B + j + i] = xhat[n * B + j + i];
  if (acc >= L || !resample) {
    if (g == 0 && tid == 0) { n_accept[n] = acc; n_commit[n] = acc; resampled[n] = -1; }
    return;
  }
  // ---- residual at block index i: r(v) = max(0, Q(v) - P(v)), both at the sampling temperature ----
  const int o = n * B + j + acc;
  const float* ld = logits_d + (size_t)row_of_d[o] * V;
  const float* lv = logits_v + (size_t)row_of_v[o] * V;
  const float zd = lse_d[o], zv = lse_v[o];
  const float u2 = uniform01(seed, stp, (uint32_t)n, (uint32_t)(j + acc), 1u);
  auto residual4 = [&](int i0, float (&r)[4]) {
    if ((V & 3) == 0) {   // unconditional loads (clamped index) so that the loads of several tiles can be in flight
      const bool ok = i0 < V;
      const int ic = ok ? i0 : 0;
      const float4 a = *(const float4*)(ld + ic), b = *(const float4*)(lv + ic);
      r[0] = ok ? fmaxf(0.f, __expf(b.x * inv_t - zv) - __expf(a.x * inv_t - zd)) : 0.f;
      r[1] = ok ? fmaxf(0.f, __expf(b.y * inv_t - zv) - __expf(a.y * inv_t - zd)) : 0.f;
      r[2] = ok ? fmaxf(0.f, __expf(b.z * inv_t - zv) - __expf(a.z * inv_t - zd)) : 0.f;
      r[3] = ok ? fmaxf(0.f, __expf(b.w * inv_t - zv) - __expf(a.w * inv_t - zd)) : 0.f;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        r[e] = (i0 + e < V) ? fmaxf(0.f, __expf(lv[i0 + e] * inv_t - zv) - __expf(ld[i0 + e] * inv_t - zd)) : 0.f;
    }
  };
  int token;
  if (G == 1) {
    token = inverse_cdf_block(residual4, V, u2, s_tile, s_w, &s_tile_sel, &s_before);
  } else {
    if (!share_tile_sums(residual4, V, g, G, tile_scratch + (size_t)n * ((V + RTILE - 1) / RTILE), &arrivals[n * ARRIVE_STRIDE], s_tile, &s_last)) return;
    token = inverse_cdf_finish(residual4, V, u2, s_tile, s_w, &s_tile_sel, &s_before);
  }
  if (tid == 0) {
    if (token < 0) token = xhat[o];  // residual without mass in fp32 (p and q equal to rounding): keep the draft
    block[o] = token;
    n_accept[n] = acc;
    n_commit[n] = acc + 1;
    resampled[n] = token;
  }
}

void launch_accept(hipStream_t st, int N, int B, int V, uint64_t seed, uint32_t step, const uint32_t* step_dev,
                   float gamma, int resample, float inv_t, const int32_t* span_start, const int32_t* span_len,
                   const float* logits_d, const int32_t* row_of_d, const float* logits_v,
                   const int32_t* row_of_v, const int32_t* xhat, const float* p, const float* lse_d,
                   const float* q, const float* lse_v, int32_t* block, int32_t* n_accept, int32_t* n_commit,
                   int32_t* resampled, float* u_used, const int32_t* active, float* tile_scratch, int32_t* arrivals) {
  // few sequences: up to 8 workgroups share the vocabulary of each (a share is then one round of the tile pass for
  // vocabularies of up to 2^18 entries)
  const int G = tile_scratch && arrivals ? std::max(1, std::min(8, 128 / N)) : 1;
  S2D2_LAUNCH(accept_kernel, dim3(N, G), dim3(1024), 0, st, B, V, seed, step, step_dev, gamma, resample, inv_t,
                     span_start, span_len, logits_d, row_of_d, logits_v, row_of_v, xhat, p, lse_d, q, lse_v, block,
                     n_accept, n_commit, resampled, u_used, active, tile_scratch, arrivals);
}

size_t tile_sum_floats(int rows, int V) { return (size_t)rows * ((V + RTILE - 1) / RTILE); }

// ---------------------------------------------------------------------------------------------
// Scratch of the accept step for callers that cannot allocate (s2d2_accept_static): the residual tile sums that
// the workgroups of a sequence hand to each other, and their arrival counters, live in a file-scope device array
// instead of the caller's workspace.  Every GPU holds its own copy of the array at its own address; the address
// is looked up once per device and only that pointer is ever passed to a kernel.
// ---------------------------------------------------------------------------------------------
static constexpr size_t STATIC_TILE_FLOATS = (size_t)ACCEPT_STATIC_MAX_BATCH * (ACCEPT_STATIC_MAX_VOCAB / RTILE);
static constexpr size_t STATIC_SCRATCH_BYTES = STATIC_TILE_FLOATS * sizeof(float) + ACCEPT_STATIC_MAX_BATCH * ARRIVE_STRIDE * sizeof(int32_t);
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];   // 544 KB per GPU, held until the process ends

static constexpr int STATIC_MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[STATIC_MAX_DEVICES];   // device address of `scratch` on each GPU, once looked up

int accept_static_scratch(float** tiles, int32_t** arrivals) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= STATIC_MAX_DEVICES) { (void)hipGetLastError(); return -1; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return -1; }
    g_scratch_ptr[dev] = ptr;
  }
  if (tiles) *tiles = (float*)g_scratch_ptr[dev];
  if (arrivals) *arrivals = (int32_t*)((unsigned char*)g_scratch_ptr[dev] + STATIC_TILE_FLOATS * sizeof(float));
  return 0;
}

}  // namespace s2d2
