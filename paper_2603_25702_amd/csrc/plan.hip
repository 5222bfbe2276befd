// Window construction and per-sequence state kernels (integer work only).
//
// plan_kernel builds, on the device and without host involvement, the packed list of window
// rows of a draft forward (block positions not yet cached, Eq. 4 visibility) or of a verifier
// forward (the 2L window of Eq. 3 with uncached committed tokens riding in front as causal
// rows).  kv_append / block_advance / commit_threshold update the per-sequence state
// (Algorithm 1 append and new block; Algorithm 2 commit).
#include "s2d2_internal.h"
#include "../../include/s2d2.h"

#include <type_traits>

namespace s2d2 {

// The token arrays live on the device and cannot be checked by the host: an id outside the vocabulary (a caller's
// mistake, or the proposal of a logit row without a single comparable value) becomes [MASK] instead of an
// embedding row outside the table.
__device__ __forceinline__ int in_vocab(int tok, int vocab, int mask_id) { return (unsigned)tok < (unsigned)vocab ? tok : mask_id; }

// Key splits of sequence n (n < N; others 0): runs of the length that gives split_target of them if all tiles were one sequence's, or of up to half as much
// more if then all splits of the batch are resident at once: the part of a run at the end of every sequence otherwise makes a few more than the
// target, and the workgroups left over start when the first ones are done.  Forwards, us, without / with: 4B draft of eight sequences of
// 1024 to 4096 tokens 4251 / 3871 (67 splits for 64), 4B verification of 20 9375 / 8788, 8B of 16 blocks behind 300 to 6000 12957 / 12284, MoE draft of 20
// 5797 / 5449.  All threads of the workgroup.
constexpr int RUNS = 16;
__device__ __forceinline__ int splits_of(int total, int tiles, int n, int N, int split_target, int split_most, int run_most, int32_t* s_runs /* [RUNS], zero */) {
  const int least = max(WIDE_MIN_TILES, (total + split_target - 1) / split_target);
  auto run = [&](int i) { return least + (least * i + 2 * RUNS - 3) / (2 * RUNS - 2); };   // least .. least * 3 / 2
  auto splits = [&](int i) { return max(1, min(split_most, (tiles + run(i) - 1) / run(i))); };
  int first = n < N ? splits(0) : 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) first += __shfl_xor(first, off, 64);
  if ((n & 63) == 0) atomicAdd(&s_runs[0], first);
  __syncthreads();
  int pick = 0;
  if (s_runs[0] > split_target) {   // uniform
    int v[RUNS];
#pragma unroll
    for (int i = 1; i < RUNS; ++i) v[i] = n < N ? splits(i) : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
      for (int i = 1; i < RUNS; ++i) v[i] += __shfl_xor(v[i], off, 64);
    if ((n & 63) == 0)
#pragma unroll
      for (int i = 1; i < RUNS; ++i) atomicAdd(&s_runs[i], v[i]);
    __syncthreads();
    for (int i = RUNS - 1; i > 0; --i)
      if (s_runs[i] <= split_target && run(i) <= run_most) pick = i;
  }
  return n < N ? splits(pick) : 0;
}

__global__ __launch_bounds__(1024) void plan_kernel(
    int verify, int shifted, int N, int B, int mask_id, int ar_mask, const int32_t* __restrict__ seq_len,
    const int32_t* __restrict__ pos0, const int32_t* __restrict__ block,
    const int32_t* __restrict__ carry, const int32_t* __restrict__ xhat, Plan p,
    int32_t* __restrict__ logit_row_of, int32_t* __restrict__ span_start,
    int32_t* __restrict__ span_len, int32_t* __restrict__ stage_row0, int32_t* __restrict__ stage_lead,
    const int32_t* __restrict__ active, int32_t* __restrict__ status, int seq_cap, int split_target, int split_most, int run_most, float* __restrict__ clear_a,
    float* __restrict__ clear_b) {
  __shared__ int32_t s_tiles, s_splits[1024], s_runs[RUNS];
  __shared__ int32_t s_rows[1024];
  __shared__ int32_t s_lrows[1024];
  const int n = threadIdx.x;
  int S = 0, c = 0, nc = 0, j = B, L = 0, n_masked = 0, rows = 0, lrows = 0, lead = 0, bad = 0;
  if (n < N) {
    S = seq_len[n];
    const int P0 = pos0[n];
    c = max(0, min(B, S - P0));
    nc = max(0, min(B, P0 - S));
    const int32_t* blk = block + (size_t)n * B;
    for (int i = 0; i < B; ++i) {
      const bool m = blk[i] == mask_id;
      n_masked += m;
      if (m && j == B) j = i;
    }
    while (j + L < B && blk[j + L] == mask_id) ++L;
    c = min(c, j);
    lead = nc + (j - c);
    if (verify == 1 && active && active[n] == 0) { L = 0; lead = 0; }   // routed to the fallback: no verifier window
    // right-shifted model: the row in front of the first [MASK] scores it and has to be a window row
    if (shifted && verify < 2 && L > 0 && lead == 0) {
      if (status) status[n] = S2D2_EINVAL;
      if (verify) L = 0;
      bad = 1;
    }
    if (verify >= 2) {            // block completion: all uncached tokens of a finished block, no logits
      rows = n_masked == 0 ? nc + (B - c) : 0;
      if (verify == 3 && rows <= B) rows = 0;   // causal variant: only what the carry list (capacity B) cannot take
      lead = rows;
      lrows = 0;
    } else if (verify) { rows = shifted ? lead + max(L - 1, 0) : lead + 2 * L; lrows = L; }
    else        { rows = nc + (B - c); lrows = bad ? 0 : n_masked; }
  }
  if (n == 0) s_tiles = 0;
  if (n < RUNS) s_runs[n] = 0;
  s_rows[n] = rows;
  s_lrows[n] = lrows;
  __syncthreads();
  // key splits: the cached key tiles of the sequences that have a window, in runs that give split_target of them
  const int tiles = rows > 0 ? (max(0, min(S, seq_cap)) + 31) >> 5 : 0;
  if (tiles) atomicAdd(&s_tiles, tiles);
  __syncthreads();
  const int splits = splits_of(s_tiles, tiles, n, N, split_target, split_most, run_most, s_runs);
  s_splits[n] = splits;
  __syncthreads();
  // inclusive Hillis-Steele scan over the sequences
  for (int off = 1; off < N; off <<= 1) {
    int a = 0, b = 0, d = 0;
    if (n >= off) { a = s_rows[n - off]; b = s_lrows[n - off]; d = s_splits[n - off]; }
    __syncthreads();
    s_rows[n] += a;
    s_lrows[n] += b;
    s_splits[n] += d;
    __syncthreads();
  }
  if (n == N - 1) { p.counts[0] = s_rows[n]; p.counts[1] = s_lrows[n]; p.counts[2] = s_splits[n]; }
  if (n >= N) return;
  const int row0 = s_rows[n] - rows;
  int k = s_lrows[n] - lrows;
  p.seq_row0[n] = row0;
  p.seq_rows[n] = rows;
  p.seq_lead[n] = lead;
  p.seq_j[n] = j;
  p.seq_L[n] = L;
  p.seq_splits[n] = splits;
  plan_write_splits(p, s_splits[n] - splits, splits, n, tiles, max(0, min(S, seq_cap)), row0, rows);
  const int32_t* blk = block + (size_t)n * B;
  const int32_t* car = carry + (size_t)n * B;
  if (!verify) {
    span_start[n] = j;
    span_len[n] = bad ? 0 : L;   // a skipped sequence has nothing to verify, accept or append
    for (int i = 0; i < B; ++i) logit_row_of[(size_t)n * B + i] = -1;
    for (int t = 0; t < rows; ++t) {
      const int r = row0 + t;
      int tok, hi;
      if (t < nc) {                       // carried token of a finished block: causal
        tok = car[t];
        hi = r + 1;
      } else {
        const int i = c + (t - nc);
        tok = blk[i];
        hi = (i < j && ar_mask) ? r + 1 : row0 + rows;   // Eq. 4: committed prefix causal, rest sees all
        if (tok == mask_id && !bad) {
          p.logit_src[k] = r - shifted;   // right-shifted model: the row in front (t >= 1 here: lead >= 1)
          p.logit_seq[k] = n;
          p.logit_idx[k] = i;
          logit_row_of[(size_t)n * B + i] = k;
          ++k;
        }
      }
      p.row_token[r] = in_vocab(tok, p.vocab, mask_id);
      p.row_pos[r] = S + t;
      p.row_seq[r] = n;
      p.row_lo[r] = row0;
      p.row_hi[r] = hi;
    }
  } else if (verify >= 2) {
    // Alg. 1 after the block sampler: carried tokens stay causal, the block's rows attend to the whole window
    // (block-diffusion attention; verify == 3: every row causal, Section 4.2); every row is staged for the cache
    stage_row0[n] = row0;
    stage_lead[n] = rows;
    for (int t = 0; t < rows; ++t) {
      const int r = row0 + t;
      p.row_token[r] = in_vocab(t < nc ? car[t] : blk[c + (t - nc)], p.vocab, mask_id);
      p.row_pos[r] = S + t;
      p.row_seq[r] = n;
      p.row_lo[r] = row0;
      p.row_hi[r] = (t < nc || verify == 3) ? r + 1 : row0 + rows;
    }
  } else {
    stage_row0[n] = row0;
    stage_lead[n] = lead;
    for (int i = 0; i < B; ++i) logit_row_of[(size_t)n * B + i] = -1;
    // per-position outputs of the verifier (q, lse) start at zero; the vocabulary pass fills the planned positions
    if (clear_a)
      for (int i = 0; i < B; ++i) { clear_a[(size_t)n * B + i] = 0.f; clear_b[(size_t)n * B + i] = 0.f; }
    const int32_t* xh = xhat + (size_t)n * B;
    const int n_drafted = shifted ? max(L - 1, 0) : L;   // a right-shifted window has no row for the last drafted token
    for (int t = 0; t < lead + n_drafted; ++t) {  // causal half: carry, pending committed, drafted C_t
      const int r = row0 + t;
      int tok;
      if (t < nc) tok = car[t];
      else if (t < lead) tok = blk[c + (t - nc)];
      else tok = xh[j + (t - lead)];
      p.row_token[r] = in_vocab(tok, p.vocab, mask_id);
      p.row_pos[r] = S + t;
      p.row_seq[r] = n;
      p.row_lo[r] = row0;
      p.row_hi[r] = r + 1;
    }
    for (int q = 0; q < L && shifted; ++q) {   // right-shifted: row of position i-1 scores the drafted token at i
      p.logit_src[k] = row0 + lead - 1 + q;
      p.logit_seq[k] = n;
      p.logit_idx[k] = j + q;
      logit_row_of[(size_t)n * B + j + q] = k;
      ++k;
    }
    for (int q = 0; q < L && !shifted; ++q) {   // [MASK] copies: see causal rows strictly left, and themselves
      const int r = row0 + lead + L + q;
      p.row_token[r] = mask_id;
      p.row_pos[r] = S + lead + q;
      p.row_seq[r] = n;
      p.row_lo[r] = row0;
      p.row_hi[r] = row0 + lead + q;
      p.logit_src[k] = r;
      p.logit_seq[k] = n;
      p.logit_idx[k] = j + q;
      logit_row_of[(size_t)n * B + j + q] = k;
      ++k;
    }
  }
}

void launch_plan(hipStream_t st, int verify, int shifted, int N, int B, int mask_id, int ar_mask,
                 const int32_t* seq_len, const int32_t* pos0, const int32_t* block,
                 const int32_t* carry, const int32_t* xhat, const Plan& p, int32_t* logit_row_of,
                 int32_t* span_start, int32_t* span_len, int32_t* stage_row0, int32_t* stage_lead,
                 const int32_t* active, int32_t* status, int seq_cap, int split_target, int split_most, int run_most, float* clear_a, float* clear_b) {
  S2D2_LAUNCH(plan_kernel, dim3(1), dim3((N + 63) / 64 * 64), 0, st, verify, shifted, N, B, mask_id, ar_mask,
                     seq_len, pos0, block, carry, xhat, p, logit_row_of, span_start, span_len,
                     stage_row0, stage_lead, active, status, seq_cap, split_target, split_most, run_most, clear_a, clear_b);
}

// Prompt tokens pushed into the cache: n_tokens[n] causal rows of sequence n behind its cached ones, no logits.  A
// wavefront fills the rows of a sequence (in plan_kernel one thread does, a few rows there, up to 192 here).
__global__ __launch_bounds__(1024) void plan_prefill_kernel(int N, int T, int mask_id, const int32_t* __restrict__ seq_len,
                                                            const int32_t* __restrict__ tokens, int ld,
                                                            const int32_t* __restrict__ n_tokens, Plan p, int seq_cap,
                                                            int split_target, int split_most, int run_most) {
  __shared__ int32_t s_tiles, s_rows[1024], s_splits[1024], s_runs[RUNS];
  const int n = threadIdx.x;
  const int S = n < N ? seq_len[n] : 0, rows = n < N ? max(0, min(T, n_tokens[n])) : 0;
  if (n == 0) s_tiles = 0;
  if (n < RUNS) s_runs[n] = 0;
  s_rows[n] = rows;
  __syncthreads();
  const int tiles = rows > 0 ? (max(0, min(S, seq_cap)) + 31) >> 5 : 0;
  if (tiles) atomicAdd(&s_tiles, tiles);
  __syncthreads();
  const int splits = splits_of(s_tiles, tiles, n, N, split_target, split_most, run_most, s_runs);
  s_splits[n] = splits;
  __syncthreads();
  for (int off = 1; off < N; off <<= 1) {
    int a = 0, d = 0;
    if (n >= off) { a = s_rows[n - off]; d = s_splits[n - off]; }
    __syncthreads();
    s_rows[n] += a;
    s_splits[n] += d;
    __syncthreads();
  }
  if (n == N - 1) { p.counts[0] = s_rows[n]; p.counts[1] = 0; p.counts[2] = s_splits[n]; }
  if (n < N) {
    p.seq_row0[n] = s_rows[n] - rows;
    p.seq_rows[n] = rows;
    p.seq_lead[n] = rows;
    p.seq_splits[n] = splits;
    plan_write_splits(p, s_splits[n] - splits, splits, n, tiles, max(0, min(S, seq_cap)), s_rows[n] - rows, rows);
  }
  for (int m = n >> 6; m < N; m += 16) {
    const int end = s_rows[m], row0 = m ? s_rows[m - 1] : 0, S0 = seq_len[m];
    for (int r = row0 + (n & 63); r < end; r += 64) {
      p.row_token[r] = in_vocab(tokens[(size_t)m * ld + (r - row0)], p.vocab, mask_id);
      p.row_pos[r] = S0 + (r - row0);
      p.row_seq[r] = m;
      p.row_lo[r] = row0;
      p.row_hi[r] = r + 1;
    }
  }
}

void launch_plan_prefill(hipStream_t st, int N, int T, int mask_id, const int32_t* seq_len, const int32_t* tokens, int ld,
                         const int32_t* n_tokens, const Plan& p, int seq_cap, int split_target, int split_most, int run_most) {
  S2D2_LAUNCH(plan_prefill_kernel, dim3(1), dim3(1024), 0, st, N, T, mask_id, seq_len, tokens, ld, n_tokens, p, seq_cap,
              split_target, split_most, run_most);
}

// ---------------------------------------------------------------------------------------------
// Cache append: copy staged K/V rows [0, lead + n_accept) of each sequence to its next logical
// positions.  One workgroup per (sequence, G consecutive slots of a page, layer).
//
// V is cached key-minor, so a row alone leaves one element in every piece of G slots; a workgroup that takes the G rows of a
// piece stores it whole, 16 bytes (the pieces at either end of the rows element by element).  Bound: the rows read and written.  768 rows of 28
// layers of 8 x 128 halves 100 -> 43 us (176 MB, 4.1 TB/s), up to 16 rows of 16 sequences in 4 layers 9.8 -> 7.1.
// ---------------------------------------------------------------------------------------------
template <typename T, int G>
__global__ __launch_bounds__(256) void kv_append_copy_kernel(
    int per_seq, int rows_cap, KvGeom g, T* __restrict__ k_pages, T* __restrict__ v_pages, const T* __restrict__ k_stage,
    const T* __restrict__ v_stage, const int32_t* __restrict__ stage_row0, const int32_t* __restrict__ stage_lead,
    const int32_t* __restrict__ n_accept, const int32_t* __restrict__ span_len, int hold_back) {
  constexpr int VE = 16 / (int)sizeof(T);
  const int n = blockIdx.x / per_seq, l = blockIdx.y;
  const int acc = max(0, min(n_accept[n], span_len[n] - hold_back));   // hold_back: no staged row for the last drafted token
  const int rows = stage_lead[n] + acc;
  const int S = g.seq_len[n];
  const int s0 = S - S % G + (blockIdx.x % per_seq) * G;   // first slot of this workgroup's piece
  if (rows <= 0 || s0 >= S + rows) return;
  const int cap = g.max_pages_per_seq * g.page_size;
  if (S + rows > cap) return;  // whole sequence skipped; the update kernel flags it
  const int page = g.page_table[(size_t)n * g.max_pages_per_seq + s0 / g.page_size];
  if (page < 0 || page >= g.n_pages) return;
  const int slot = s0 % g.page_size, D = g.head_dim, HD = g.n_kv_heads * D;
  const int u0 = max(0, S - s0), u1 = min(G, S + rows - s0);   // places of the piece that are written
  const size_t src = ((size_t)l * rows_cap + stage_row0[n]) * HD;
  const int t0 = s0 - S;                                       // staged row of place 0
  const size_t page_off = ((size_t)l * g.n_pages + page) * HD * g.page_size;
  const int vecs = HD / VE;   // 16-byte pieces of a staged row
  for (int v = threadIdx.x; v < (u1 - u0) * vecs; v += 256) {
    const int u = u0 + v / vecs, e = (v % vecs) * VE, h = e / D;
    *(uint4*)(k_pages + page_off + ((size_t)h * g.page_size + slot + u) * D + e % D) = *(const uint4*)(k_stage + src + (size_t)(t0 + u) * HD + e);
  }
  // V is cached key-minor: [page, Hkv, D, page_size]; two elements of the head dimension per thread
  for (int v = threadIdx.x * 2; v < HD; v += 512) {
    alignas(16) T lo[G], hi[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      struct alignas(2 * sizeof(T)) Pair { T a, b; };
      const Pair x = *(const Pair*)(v_stage + src + (size_t)(t0 + min(max(u, u0), u1 - 1)) * HD + v);   // (a place that is not written reads one that is)
      lo[u] = x.a;
      hi[u] = x.b;
    }
    T* dst = v_pages + page_off + (size_t)v * g.page_size + slot;
    if (G * sizeof(T) == 16 && u0 == 0 && u1 == G) {
      *(uint4*)dst = *(const uint4*)lo;
      *(uint4*)(dst + g.page_size) = *(const uint4*)hi;
    } else {
#pragma unroll
      for (int u = 0; u < G; ++u)
        if (u >= u0 && u < u1) {
          dst[u] = lo[u];
          dst[g.page_size + u] = hi[u];
        }
    }
  }
}

__global__ void kv_append_commit_kernel(int N, KvGeom g, const int32_t* __restrict__ stage_lead,
                                        const int32_t* __restrict__ n_accept,
                                        const int32_t* __restrict__ span_len, int32_t* __restrict__ seq_len,
                                        int32_t* __restrict__ status, int hold_back) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int acc = max(0, min(n_accept[n], span_len[n] - hold_back));
  const int rows = stage_lead[n] + acc;
  const int S = seq_len[n];
  if (S + rows > g.max_pages_per_seq * g.page_size) {
    if (status) status[n] = S2D2_ENOSPC;
    return;
  }
  seq_len[n] = S + rows;
}

void launch_kv_append(hipStream_t st, int dtype, int n_layers, int N, int rows_cap, const KvGeom& g,
                      void* k_pages, void* v_pages, const void* k_stage, const void* v_stage,
                      const int32_t* stage_row0, const int32_t* stage_lead, const int32_t* span_len,
                      const int32_t* n_accept, int32_t* seq_len, int32_t* status, int B, int hold_back) {
  // 2 B: upper bound of staged causal rows per sequence (carry + block); pieces of whole 16 bytes where no page cuts one
  auto copy = [&](auto elt, auto group) {
    using T = decltype(elt);
    constexpr int G = decltype(group)::value;
    const int per_seq = (2 * B + G - 2) / G + 1;   // rows may begin inside a piece
    S2D2_LAUNCH((kv_append_copy_kernel<T, G>), dim3(N * per_seq, n_layers), dim3(256), 0, st, per_seq, rows_cap, g, (T*)k_pages, (T*)v_pages,
                (const T*)k_stage, (const T*)v_stage, stage_row0, stage_lead, n_accept, span_len, hold_back);
  };
  if (dtype == S2D2_BF16) {
    if (g.page_size % 8 == 0) copy(uint16_t{}, std::integral_constant<int, 8>{}); else copy(uint16_t{}, std::integral_constant<int, 1>{});
  } else {
    if (g.page_size % 4 == 0) copy(uint32_t{}, std::integral_constant<int, 4>{}); else copy(uint32_t{}, std::integral_constant<int, 1>{});
  }
  S2D2_LAUNCH(kv_append_commit_kernel, dim3((N + 255) / 256), dim3(256), 0, st, N, g, stage_lead,
                     n_accept, span_len, seq_len, status, hold_back);
}

// ---------------------------------------------------------------------------------------------
// Alg. 1: replace a block that holds no [MASK] by a fresh [MASK]^B block right after it.
// Uncached committed tokens of the finished block move to the carry list (capacity B); if they
// would not fit, the block is left as it is and the sequence's status word says so (the caller
// caches them first: s2d2_block_complete).
// ---------------------------------------------------------------------------------------------
__global__ void block_advance_kernel(int N, int B, int mask_id, const int32_t* __restrict__ seq_len,
                                     int32_t* __restrict__ pos0, int32_t* __restrict__ block,
                                     int32_t* __restrict__ carry, uint32_t* step_dev, int32_t* __restrict__ status) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n == 0 && step_dev) *step_dev += 1u;
  if (n >= N) return;
  int32_t* blk = block + (size_t)n * B;
  int32_t* car = carry + (size_t)n * B;
  for (int i = 0; i < B; ++i)
    if (blk[i] == mask_id) return;
  const int S = seq_len[n], P0 = pos0[n];
  const int c = max(0, min(B, S - P0)), nc = max(0, min(B, P0 - S));
  if (nc + (B - c) > B) {
    if (status) status[n] = S2D2_ENOSPC;
    return;
  }
  for (int i = c; i < B; ++i) car[nc + (i - c)] = blk[i];
  for (int i = 0; i < B; ++i) blk[i] = mask_id;
  pos0[n] = P0 + B;
}

void launch_block_advance(hipStream_t st, int N, int B, int mask_id, const int32_t* seq_len,
                          int32_t* pos0, int32_t* block, int32_t* carry, uint32_t* step_dev, int32_t* status) {
  S2D2_LAUNCH(block_advance_kernel, dim3((N + 255) / 256), dim3(256), 0, st, N, B, mask_id, seq_len,
                     pos0, block, carry, step_dev, status);
}

__global__ void commit_threshold_kernel(int N, int B, int32_t* __restrict__ block,
                                        const int32_t* __restrict__ xhat, const uint64_t* __restrict__ unmask) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= N * B) return;
  const int n = idx / B, i = idx % B;
  if ((unmask[n] >> i) & 1ull) block[idx] = xhat[idx];
}

void launch_commit_threshold(hipStream_t st, int N, int B, int32_t* block, const int32_t* xhat,
                             const uint64_t* unmask) {
  S2D2_LAUNCH(commit_threshold_kernel, dim3((N * B + 255) / 256), dim3(256), 0, st, N, B, block, xhat,
                     unmask);
}

// ---------------------------------------------------------------------------------------------
// Verification routing (Section 4.3): one thread per sequence.  K = sum_k prod_{i<=k} alpha_i over C_t,
// score, policy decision, hysteresis state update.
// ---------------------------------------------------------------------------------------------
__global__ void route_kernel(int N, int B, s2d2_route_params rp, const int32_t* __restrict__ span_start,
                             const int32_t* __restrict__ span_len, const float* __restrict__ margin,
                             const float* __restrict__ entropy_n, const int32_t* __restrict__ n_hi,
                             const uint64_t* __restrict__ unmask, int32_t* __restrict__ hysteresis,
                             int32_t* __restrict__ do_verify, float* __restrict__ khat, float* __restrict__ score,
                             uint64_t* __restrict__ unmask_fallback) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int j = span_start[n], L = max(0, min(span_len[n], B - j));
  float prod = 1.f, k = 0.f;
  for (int i = 0; i < L; ++i) {
    const int o = n * B + j + i;
    const float a = rp.estimator == S2D2_EST_MARGIN ? (margin[o] >= rp.tau_margin ? 1.f : 0.f)
                                                    : expf(-rp.beta * entropy_n[o]);
    prod *= a;
    k += prod;
  }
  const float s = rp.dynamic ? k - rp.c * (float)n_hi[n] : k - rp.c;
  bool dec;
  if (rp.policy == S2D2_ROUTE_MIN_SPAN) {
    dec = L >= rp.tau_span;
  } else if (rp.policy == S2D2_ROUTE_SCORE) {
    dec = s >= rp.tau_score;
  } else {
    int h = hysteresis[n] != 0;
    if (L > 0) {   // a block without a masked span leaves the state as it is
      if (h && s < rp.tau_off) h = 0;
      else if (!h && s >= rp.tau_on) h = 1;
      hysteresis[n] = h;
    }
    dec = h != 0;
  }
  dec = dec && L > 0;
  do_verify[n] = dec ? 1 : 0;
  khat[n] = k;
  score[n] = s;
  unmask_fallback[n] = dec ? 0ull : unmask[n];
}

void launch_route(hipStream_t st, int N, int B, const s2d2_route_params& rp, const int32_t* span_start,
                  const int32_t* span_len, const float* margin, const float* entropy_n, const int32_t* n_hi,
                  const uint64_t* unmask, int32_t* hysteresis, int32_t* do_verify, float* khat, float* score,
                  uint64_t* unmask_fallback) {
  S2D2_LAUNCH(route_kernel, dim3((N + 255) / 256), dim3(256), 0, st, N, B, rp, span_start, span_len, margin,
              entropy_n, n_hi, unmask, hysteresis, do_verify, khat, score, unmask_fallback);
}

}  // namespace s2d2
