// Attention of one window row over the paged prefix cache plus the visible in-window keys.
//
// attn_generic_kernel: plain fp32 arithmetic, one workgroup per (window row, query head).  It is
// the reference-quality path (used for fp32 models and as the cross-check of the MFMA kernel):
// scores of all keys go to LDS, a block-wide softmax follows, then P*V with the head dimension
// across lanes.  Visibility inside the window follows the plan (Eq. 3 / Eq. 4): window row w is
// visible to row r iff row_lo[r] <= w < row_hi[r] or w == r; every cached position is visible.
#include "s2d2_internal.h"
#include "../../include/s2d2.h"
#include "attention_flash.h"

namespace s2d2 {

template <int I> struct Lane { static constexpr int value = I; };

__device__ __forceinline__ float wave_max(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Every sum has one association, whatever the batch and the cache size are: a score is one chain over the head dimension,
// the softmax denominator the sum of 256 strided ones, P V 256 / D chains of every (256 / D)-th key.  (With four partial
// scores a key, 1024 / D chains and 1024 strided sums where LDS had room for that many threads, the results were as close
// to 64 bits, but a sequence's own depended on the capacity of the cache it sat in: its logits by 5e-7 of their norm, its
// margins, differences of two nearly equal probabilities, by up to 8e-5.)
//
// The launch is a chain of round trips to memory, so its 1024 threads request what they can at once and hand the chains
// on: four lanes take 16 bytes of a key's row each, in turn; P V runs through four quarters of the workgroup, VB keys of
// a chain each, whose V values are requested ahead of the scores.  8 and 12 rows over 136 keys of 64 floats: 10.6 and
// 11.3 us per launch (12.9 and 13.4 with the page look-ups under a condition: each was waited for); 256 threads with a key
// each and one V value per iteration took 16.8.
template <typename T, int D>
__global__ __launch_bounds__(1024) void attn_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ k_win, const T* __restrict__ v_win,
    const T* __restrict__ k_pages, const T* __restrict__ v_pages, KvGeom g, Plan p, int Hq,
    T* __restrict__ o, float scale, int o_lo) {
  constexpr int NT = 1024, VE = 16 / (int)sizeof(T), NCH = D / (4 * VE), CB = NCH < 4 ? NCH : 4;   // NCH: 16-byte pieces of a row per lane, CB: requested at once
  constexpr int NS = 256 / D, VB = 12;
  extern __shared__ float smem[];
  const int r = blockIdx.x, hq = blockIdx.y;
  if (r >= p.counts[0]) return;
  const int Hkv = g.n_kv_heads, ps = g.page_size;
  const int kvh = hq / (Hq / Hkv);
  const int n = p.row_seq[r];
  const int S = max(0, min(g.seq_len[n], g.max_pages_per_seq * ps));
  const int row0 = p.seq_row0[n], nw = p.seq_rows[n];
  const int lo = p.row_lo[r], hi = p.row_hi[r];
  const int total = S + nw;
  float* s_q = smem;             // [D]
  float* s_red = smem + D;       // [256 + 8]
  float* s_sc = s_red + 264;     // [total]
  const int tid = threadIdx.x, wave = tid >> 6;
  const int32_t* pt = g.page_table + (size_t)n * g.max_pages_per_seq;

  // Requests in the order in which they are needed (loads return in order): the query, the page of this lane's first key, the
  // pages of the first V values, the key, the V values.  Behind the query's store to LDS only those are in flight.
  const float q0 = tid < D ? to_f32(q[((size_t)r * Hq + hq) * D + tid]) : 0.f;
  const int part = tid & 3, quarter = tid >> 8, t8 = tid & 255, d = t8 % D, sl = t8 / D;
  // Places in the cache: division by a page size that is a power of two is a shift (thirteen divisions per thread are a fifth of the launch's instructions), and
  // a block's number (n_pages Hkv) fits 32 bits, as a block is 128 bytes or more.
  const bool p2 = (ps & (ps - 1)) == 0;
  const int sh = 31 - __builtin_clz(ps);
  const uint32_t block = (uint32_t)ps * D;
  auto cached_at = [&](int s) __attribute__((always_inline)) { return max(min(s, S - 1), 0); };   // (without cached keys the first page is looked up all the same: a load under a condition is waited for before the next one)
  auto place = [&](int s, int& page, int& slot) __attribute__((always_inline)) {
    const int c = cached_at(s);
    int i;
    if (p2) i = c >> sh;
    else i = c / ps;
    page = pt[i];
    slot = c - i * ps;
  };
  auto page0 = [&](int page) __attribute__((always_inline)) { return (uint64_t)((uint32_t)min(max(page, 0), g.n_pages - 1) * (uint32_t)Hkv + kvh) * block; };
  auto win0 = [&](int s) __attribute__((always_inline)) { return (uint64_t)((uint32_t)(row0 + max(s - S, 0)) * (uint32_t)Hkv + kvh) * (uint32_t)D; };
  auto key_row = [&](int s, int page, int slot) __attribute__((always_inline)) {
    const T* cached = k_pages + page0(page) + (uint32_t)slot * (uint32_t)D;
    const T* own = k_win + win0(s);
    return s < S ? cached : own;
  };
  uint4 kv[CB];   // pieces of the key's row that this lane adds next
  auto load_k = [&](const T* kp, int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < CB; ++c) kv[c] = *(const uint4*)(kp + ((c0 + c) * 4 + part) * VE);
  };
  // V values of the keys at places e0 + VB quarter .. of this thread's chain (key = slice + NS place; past the end the last key)
  T val[VB];
  int vpage[VB], vslot[VB];
  auto key_of = [&](int e0, int u) __attribute__((always_inline)) { return sl + (e0 + quarter * VB + u) * NS; };
  auto find_v = [&](int e0) __attribute__((always_inline)) {
    if (p2) {
#pragma unroll
      for (int u = 0; u < VB; ++u) vpage[u] = cached_at(key_of(e0, u)) >> sh;
    } else {
#pragma unroll
      for (int u = 0; u < VB; ++u) vpage[u] = cached_at(key_of(e0, u)) / ps;
    }
#pragma unroll
    for (int u = 0; u < VB; ++u) {
      vslot[u] = cached_at(key_of(e0, u)) - vpage[u] * ps;
      vpage[u] = pt[vpage[u]];
    }
  };
  auto load_v = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < VB; ++u) {
      const int s = min(key_of(e0, u), total - 1);
      const T* cached = v_pages + page0(vpage[u]) + (uint32_t)(d * ps + vslot[u]);   // cache V is stored [D, page_size]
      const T* own = v_win + win0(s) + (uint32_t)d;
      val[u] = *(s < S ? cached : own);
    }
  };
  const int first = min(tid >> 2, total - 1);
  int kpage, kslot;
  place(first, kpage, kslot);
  find_v(0);
  load_k(key_row(first, kpage, kslot), 0);
  load_v(0);
  if (tid < D) s_q[tid] = q0 * scale;
  __syncthreads();

  float lmax = -INFINITY;
  for (int s0 = 0; s0 < total; s0 += NT / 4) {
    const int s = min(s0 + (tid >> 2), total - 1), w = row0 + (s - S);
    const bool vis = s < S || (w >= lo && w < hi) || w == r;
    if (s0) place(s, kpage, kslot);
    const T* kp = key_row(s, kpage, kslot);
    float dot = 0.f;   // the same in all four lanes of the key
#pragma unroll
    for (int c0 = 0; c0 < NCH; c0 += CB) {
      if (s0 || c0) load_k(kp, c0);
#pragma unroll
      for (int c = 0; c < CB; ++c) {
        const T* e = (const T*)&kv[c];
        const float* qe = s_q + ((c0 + c) * 4 + part) * VE;
        float qv[VE];
#pragma unroll
        for (int i = 0; i < VE; ++i) qv[i] = qe[i];
        auto turn = [&](auto P) __attribute__((always_inline)) {   // lane P of the four adds its piece and passes the sum on
          float t = dot;
#pragma unroll
          for (int i = 0; i < VE; ++i) t = __builtin_fmaf(qv[i], to_f32(e[i]), t);
          dot = __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(t), decltype(P)::value * 0x55, 0xf, 0xf, true));
        };
        turn(Lane<0>{}); turn(Lane<1>{}); turn(Lane<2>{}); turn(Lane<3>{});
      }
    }
    if (!vis) dot = -INFINITY;
    if (part == 0 && s0 + (tid >> 2) < total) s_sc[s] = dot;
    lmax = fmaxf(lmax, dot);
  }
  lmax = wave_max(lmax);
  if ((tid & 63) == 0) s_red[wave] = lmax;
  __syncthreads();
  float m = s_red[0];
  for (int w = 1; w < NT / 64; ++w) m = fmaxf(m, s_red[w]);
  __syncthreads();
  if (tid < 256) {
    float lsum = 0.f;
    for (int s = tid; s < total; s += 256) {
      const float e = __expf(s_sc[s] - m);   // exp(-inf) = 0 for invisible keys
      s_sc[s] = e;
      lsum += e;
    }
    lsum = wave_sum(lsum);
    if ((tid & 63) == 0) s_red[wave] = lsum;
  }
  __syncthreads();
  const float denom = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
  __syncthreads();

  for (int e0 = 0; e0 * NS < total; e0 += 4 * VB) {
    if (e0) { find_v(e0); load_v(e0); }
    float pw[VB];
#pragma unroll
    for (int u = 0; u < VB; ++u) pw[u] = key_of(e0, u) < total ? s_sc[key_of(e0, u)] : 0.f;
    for (int w = 0; w < 4; ++w) {
      if (quarter == w) {
        float acc = e0 + w ? s_red[t8] : 0.f;
#pragma unroll
        for (int u = 0; u < VB; ++u) {
          const float t = __builtin_fmaf(pw[u], to_f32(val[u]), acc);
          acc = pw[u] != 0.f ? t : acc;   // (an invisible key adds nothing, whatever its value is)
        }
        s_red[t8] = acc;
      }
      __syncthreads();
    }
  }
  if (tid < D) {
    float t = 0.f;
    for (int i = 0; i < NS; ++i) t += s_red[i * D + tid];
    if (sizeof(T) == 2 && o_lo < 0) ((bf16_t*)o)[act_offset(o_lo, r, hq * D + tid, Hq * D)] = f32_to_f16_bits(t / denom);   // the consuming GEMM runs on half operands
    else o[((size_t)r * Hq + hq) * D + tid] = from_f32<T>(t / denom);
  }
}

template <int NW, bool SPLIT>
__global__ __launch_bounds__(NW * 64) void attn_flash_kernel(
    const bf16_t* __restrict__ q, int q_ld, int q_lo, const bf16_t* __restrict__ k_win, const bf16_t* __restrict__ vT_win,
    const bf16_t* __restrict__ k_pages, const bf16_t* __restrict__ v_pages, KvGeom g, Plan p, int Hq, int Z,
    int wpad, float scale_log2e, bf16_t* __restrict__ o, int o_ld, int o_lo, float* __restrict__ part_o,
    float* __restrict__ part_ml, int32_t* __restrict__ counters, int items, const uint4* __restrict__ pf, size_t pf_n16) {
  extern __shared__ float smem[];
  if ((int)blockIdx.z >= items) {
    // Workgroups behind the attention's own: they read the weights of the GEMMs that follow this launch, so that
    // those find them in the memory-side cache.  The attention is bound by dependent round trips, not by
    // bandwidth, and leaves most compute units and nearly all of the HBM time of its launch unused.
    const size_t nwg = (size_t)(gridDim.z - items) * gridDim.y * gridDim.x;
    const size_t wg = ((size_t)(blockIdx.z - items) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const size_t per = (pf_n16 + nwg - 1) / nwg, b0 = wg * per, b1 = min(pf_n16, b0 + per);
    for (size_t i = b0 + threadIdx.x; i < b1; i += (size_t)8 * NW * 64) {
      uint4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = pf[min(i + (size_t)u * NW * 64, b1 - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(v[u].x), "v"(v[u].y), "v"(v[u].z), "v"(v[u].w));
    }
    return;
  }
  attn_flash_body<NW, SPLIT, false>(q, q_ld, q_lo, k_win, vT_win, k_pages, v_pages, g, p, Hq, Z, wpad, scale_log2e, o, o_ld,
                                    o_lo, part_o, part_ml, counters, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y, smem);
}


// Floats needed for `entries` split partials (one per (sequence, KV head, query tile, split)).
size_t attention_flash_partial_floats(size_t entries) { return entries * (32 * FA_D + 64); }

// q_tiles = ceil(3 B grp / 32); Z key splits of 8 wavefronts each.  `counters` holds one zeroed
// arrival counter per (sequence, KV head, query tile); the last split to arrive merges.
void launch_attention_flash(hipStream_t st, const void* q, int q_ld, int q_lo, const void* k_win, const void* vT_win,
                            const void* k_pages_layer, const void* v_pages_layer, const KvGeom& g, const Plan& p,
                            int N, int Hq, int q_tiles, int Z, int wpad, void* o, int o_ld, int o_lo, float* part,
                            int32_t* counters, const void* prefetch, size_t prefetch_bytes, int prefetch_wgs) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)g.head_dim);
  const int items = N * g.n_kv_heads;
  float* part_o = part;
  float* part_ml = part + (size_t)items * q_tiles * Z * 32 * FA_D;
  // extra slabs of Z * q_tiles workgroups that only read `prefetch` (see the kernel)
  const int slabs = prefetch && prefetch_bytes >= 16 ? std::min(65535 - items, (prefetch_wgs + Z * q_tiles - 1) / (Z * q_tiles)) : 0;
  const uint4* pf = (const uint4*)prefetch;
  const size_t pf_n16 = slabs > 0 ? prefetch_bytes / 16 : 0;
  if (q_lo)
    S2D2_LAUNCH((attn_flash_kernel<8, true>), dim3(Z, q_tiles, items + slabs), dim3(8 * 64), fa_lds(8), st,
                       (const bf16_t*)q, q_ld, q_lo, (const bf16_t*)k_win, (const bf16_t*)vT_win,
                       (const bf16_t*)k_pages_layer, (const bf16_t*)v_pages_layer, g, p, Hq, Z, wpad, scale_log2e,
                       (bf16_t*)o, o_ld, o_lo, part_o, part_ml, counters, items, pf, pf_n16);
  else
    S2D2_LAUNCH((attn_flash_kernel<8, false>), dim3(Z, q_tiles, items + slabs), dim3(8 * 64), fa_lds(8), st,
                       (const bf16_t*)q, q_ld, q_lo, (const bf16_t*)k_win, (const bf16_t*)vT_win,
                       (const bf16_t*)k_pages_layer, (const bf16_t*)v_pages_layer, g, p, Hq, Z, wpad, scale_log2e,
                       (bf16_t*)o, o_ld, o_lo, part_o, part_ml, counters, items, pf, pf_n16);
}

#ifdef S2D2_KERNEL_TIMING
__global__ void attn_ts_copy_kernel(unsigned long long* out) { if (threadIdx.x < 64) out[threadIdx.x] = g_attn_ts[threadIdx.x]; }
void launch_attn_ts_copy(hipStream_t st, void* out) { S2D2_LAUNCH(attn_ts_copy_kernel, dim3(1), dim3(64), 0, st, (unsigned long long*)out); }
#else
void launch_attn_ts_copy(hipStream_t, void*) {}
#endif

__global__ void fill_i32_kernel(int32_t* p, int n, int32_t v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
void launch_fill_i32(hipStream_t st, int32_t* p, int n, int32_t v) {
  S2D2_LAUNCH(fill_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
}

// Raises the dynamic-LDS limit of the kernels once (160 KB per workgroup on gfx950).
int attention_init() {
  hipError_t e = hipSuccess;
  auto limit = [&](const void* f) { if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024); };
  limit((const void*)attn_generic_kernel<bf16_t, 32>); limit((const void*)attn_generic_kernel<float, 32>);
  limit((const void*)attn_generic_kernel<bf16_t, 64>); limit((const void*)attn_generic_kernel<float, 64>);
  limit((const void*)attn_generic_kernel<bf16_t, 128>); limit((const void*)attn_generic_kernel<float, 128>);
  limit((const void*)attn_generic_kernel<bf16_t, 256>); limit((const void*)attn_generic_kernel<float, 256>);
  if (e == hipSuccess) e = hipFuncSetAttribute((const void*)attn_flash_kernel<8, false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fa_lds(8));
  if (e == hipSuccess) e = hipFuncSetAttribute((const void*)attn_flash_kernel<8, true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)fa_lds(8));
  return e == hipSuccess ? 0 : -1;
}

size_t attention_generic_lds_bytes(const KvGeom& g, int max_window_rows) {
  const size_t keys = (size_t)g.max_pages_per_seq * g.page_size + max_window_rows;
  return (g.head_dim + 264 + keys) * sizeof(float);
}

template <typename T, int D>
static void launch_generic(hipStream_t st, const void* q, const void* k_win, const void* v_win, const void* k_pages, const void* v_pages,
                           const KvGeom& g, const Plan& p, int rows_cap, int Hq, void* o, size_t lds_bytes, int o_lo) {
  S2D2_LAUNCH((attn_generic_kernel<T, D>), dim3(rows_cap, Hq), dim3(1024), lds_bytes, st, (const T*)q, (const T*)k_win, (const T*)v_win,
              (const T*)k_pages, (const T*)v_pages, g, p, Hq, (T*)o, 1.0f / sqrtf((float)D), o_lo);
}

void launch_attention_generic(hipStream_t st, int dtype, const void* q, const void* k_win, const void* v_win,
                              const void* k_pages_layer, const void* v_pages_layer, const KvGeom& g,
                              const Plan& p, int rows_cap, int Hq, void* o, size_t lds_bytes, int o_lo) {
#define S2D2_GENERIC(DV)                                                                                                          \
  case DV:                                                                                                                        \
    if (dtype == S2D2_BF16) launch_generic<bf16_t, DV>(st, q, k_win, v_win, k_pages_layer, v_pages_layer, g, p, rows_cap, Hq, o, lds_bytes, o_lo); \
    else launch_generic<float, DV>(st, q, k_win, v_win, k_pages_layer, v_pages_layer, g, p, rows_cap, Hq, o, lds_bytes, 0);       \
    break
  switch (g.head_dim) {   // (the description's check admits no others)
    S2D2_GENERIC(32);
    S2D2_GENERIC(64);
    S2D2_GENERIC(128);
    S2D2_GENERIC(256);
  }
#undef S2D2_GENERIC
}

}  // namespace s2d2
