// Flash attention for windows with several 32-row query tiles (batched verification, large blocks).
//
// attn_flash_kernel gives every query tile a workgroup of its own, so a (sequence, KV head) pair with
// q_tiles query tiles reads its cached K / V q_tiles times.  Here the NW wavefronts of a workgroup each own
// ONE query tile of the same (sequence, KV head, key split) and walk the keys together: a 32-key tile of K
// and of V^T is fetched from global memory once per workgroup, parked in LDS, and read from there as MFMA operands by all
// wavefronts.  Key splits are added up by a second launch, in split order.
//
// Eight wavefronts (one workgroup per compute unit) of which at most half have a query tile with rows, as in every window without
// committed tokens in front: in splits of more than FW_SHORT tiles they stand in two key groups, the group of an even and of an odd
// tile, so a step of the walk is two tiles long and every wavefront multiplies; the two states of a query tile are merged in LDS at the end.
// In shorter splits, and beside a page table that leaves no LDS for four tiles, the lower four multiply and the upper four fetch, one tile at a time, with plain loads: what two groups
// save over a few tiles is less than their merge and the streaming loads' longer way cost.
//
// Pipeline: two groups of tiles are in flight in registers while a third is being consumed from one of two LDS buffers; a
// wavefront parks its pieces of group g + 1 in the other buffer after its own math on group g, and one barrier per group
// separates that from the reads of group g + 1.  The page-table entries of the split's key range are copied to LDS
// once, and read a group ahead of the loads that need them.  What bounds a long prefix is the issue of vector-ALU
// instructions (softmax, conversions, addresses), then the clock, which falls to 1.7 .. 1.9 GHz here.
// Attention per launch (without the merge), one tile at a time with separate fetching wavefronts / two tiles in two key groups:
// 8B verification, 32 sequences of 2048 .. 8192 tokens 141 / 113 us.
#include "attention_flash.h"
#include <stdlib.h>
#include <type_traits>

namespace s2d2 {

#ifdef S2D2_KERNEL_TIMING
__device__ unsigned long long g_wide_ts[64];
// stamps of the first wavefront of workgroup (0, 0, 0), tile 16
#define S2D2_WTS(k, cond) do { if ((cond) && lane == 0 && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0) g_wide_ts[(k)] = wall_clock64(); } while (0)
__global__ void wide_ts_copy_kernel(unsigned long long* out) { if (threadIdx.x < 64) out[threadIdx.x] = g_wide_ts[threadIdx.x]; }
void launch_wide_ts_copy(hipStream_t st, void* out) { S2D2_LAUNCH(wide_ts_copy_kernel, dim3(1), dim3(64), 0, st, (unsigned long long*)out); }
#else
#define S2D2_WTS(k, cond) do {} while (0)
void launch_wide_ts_copy(hipStream_t, void*) {}
#endif

static constexpr int FW_KROW = 272;               // bytes per K row in LDS: 128 bf16 + 16 bytes (bank spread)
static constexpr int FW_VROW = 80;                // bytes per V^T row in LDS: 32 keys bf16 + 16 bytes
static constexpr int FW_KBUF = 32 * FW_KROW;
static constexpr int FW_BUF = FW_KBUF + 128 * FW_VROW;
static constexpr int FW_RING = 2;
// Tiles up to which four of eight wavefronts fetch for the others (see the header).  us per launch with the merge, fetching / two key
// groups: 5 tiles 4B draft 2 x 32 behind 1000 16.3 / 18.5 (two planes 20.3 / 21.8), MoE 4 x 16 17.1 / 20.0, 8 tiles 4B 21.6 / 23.6, 17 tiles 8B
// 16 x 16 31.0 / 34.5, 25 tiles 8B 16 x 16 37.0 / 39.1, 8 x 16 36.6 / 36.2, 33 tiles 8 x 16 41.5 / 41.4, 129 tiles 16 x 16 126 / 115.
static constexpr int FW_SHORT = 24;
// Tiles up to which workgroups of four wavefronts load past no cache, in launches of more workgroups than compute units.  Launches, plain /
// streaming loads, us with the merge: 4 tiles 8B verification 1 x 5 behind 6000 20.6 / 22.8, 1.7B 5 x 7 behind 300 to 1900 18.8 / 20.9, 4B draft
// 4 x 16 behind 1000 17.3 / 18.1, 6 tiles 23.9 / 25.6, 12 tiles 32.2 / 33.0, 16 tiles 8B 16 x 16 40.2 / 39.3, 4B 8 x 8 34.8 / 33.3, 24 tiles 4 x 16
// 49.3 / 47.4, 64 tiles 8B 16 x 16 110 / 99.5.  Whole forwards, streaming / plain: 376 workgroups (the 8B one) 3909 / 3866, 360 (the 1.7B one)
// 1976 / 1964, 384 4B 2 x 9 behind 3000 3394 / 3396, 8B 3 x 5 behind 2000 4224 / 4230; but 136 1.7B 3 x 10 behind 700 1883 / 1933, 64 1.7B
// 2 x 10 behind 320 1629 / 1637.
static constexpr int FW_SHORT4 = 8;

size_t attention_wide_lds_bytes(int pt_cap, int tiles) { return (size_t)FW_RING * tiles * FW_BUF + (size_t)pt_cap * 4; }

struct FwTile { bool win; int kbase, limit; };

// Keeps the first nv of 8 bf16 and zeroes the rest, without branches.
__device__ __forceinline__ uint4 fw_mask(uint4 v, int nv) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int k = nv - 2 * e;   // valid halves of this dword
    const uint32_t m = k >= 2 ? 0xffffffffu : (k == 1 ? 0xffffu : 0u);
    w[e] &= m;
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// (Every byte of the cache is read once per launch.  STREAM: past the caches, 7.0 TB/s for the 6.1 of plain loads in a long walk; a short one
// ends sooner with plain loads, see FW_SHORT4.)
template <bool STREAM>
__device__ __forceinline__ uint4 ld_kv(uint64_t at) {
  if (!STREAM) return __builtin_bit_cast(uint4, *(const __attribute__((address_space(1))) u32x4_t*)at);
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4_t*)at));
}

// 8 bf16 values (one 16-byte operand piece) as IEEE half: exact for magnitudes in the half range (the 8-bit
// significand fits), values below 2^-14 land on half subnormals (absolute error below 2^-24).
__device__ __forceinline__ uint32_t fw_bf16x2_to_f16x2(uint32_t w) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u)));
}
__device__ __forceinline__ uint4 fw_to_f16(uint4 v) {
  return make_uint4(fw_bf16x2_to_f16x2(v.x), fw_bf16x2_to_f16x2(v.y), fw_bf16x2_to_f16x2(v.z), fw_bf16x2_to_f16x2(v.w));
}

// QM: how the queries come and the arithmetic type of both products.  OPM_BF16 / OPM_BF16X2: bf16 MFMA on the
// cache's bf16 keys and values, queries and softmax weights as one or as a high + low bf16 plane.  OPM_F16: queries
// as IEEE half, keys and values converted to half on their way into LDS, softmax
// weights as half: one 11-bit plane on the f16 MFMA, half the matrix instructions of the two-plane form and no
// high / low split of the weights.
template <int NW, int QM>
__global__ __launch_bounds__(NW * 64, 2) void attn_flash_wide_kernel(
    const bf16_t* __restrict__ q, int q_ld, int q_lo, const bf16_t* __restrict__ k_win, const bf16_t* __restrict__ vT_win,
    const bf16_t* __restrict__ k_pages, const bf16_t* __restrict__ v_pages, KvGeom g, Plan p, int Hq, int Z,
    int wpad, float scale_log2e, bf16_t* __restrict__ o, int o_ld, int o_lo, float* __restrict__ part_o,
    float* __restrict__ part_ml, int q_tiles, int per, int pt_cap, int ps_shift, int tiles /* there is LDS for */, int cus) {
  constexpr int D = FA_D, T = NW * 64;
  constexpr bool SPLIT = QM == OPM_BF16X2, F16 = QM == OPM_F16;
  extern __shared__ __align__(16) unsigned char lds[];
  int32_t* s_pt = (int32_t*)(lds + FW_RING * tiles * FW_BUF);
  // Splits are numbered through over the sequences (Plan.split_of), so the workgroups without one are the last of the
  // grid.  Between the others they leave compute units empty that hold two workgroups elsewhere, one after the
  // other (the hardware deals workgroups out in turn, whether they leave at once or not): 125 -> 167 us.
  const int qgrp = blockIdx.y;
  const int4 so = p.split_of[2 * blockIdx.z], sq = p.split_of[2 * blockIdx.z + 1];   // (one round trip for all of a split's description)
  const int n_splits = p.counts[2];
  if ((int)blockIdx.z >= n_splits) return;
  const int n = so.x, z = so.y, t0 = so.z, t1 = so.w, Zn = sq.x, S = sq.y, row0 = sq.z, nw = sq.w;
  const int Hkv = g.n_kv_heads, ps = g.page_size;
  const int kvh = blockIdx.x, item = n * Hkv + kvh;
  const int grp = Hq / Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int cap = g.max_pages_per_seq * ps;
  const int nq = nw * grp;
  // query tiles qgrp * per .. + per of this (sequence, KV head) belong to this workgroup, one per wavefront (per <= NW)
  if (qgrp * per * 32 >= nq) return;            // the whole workgroup: nothing to do (before any barrier)
  // Query tiles with rows; see the header for what at least two of eight wavefronts for each are used for.
  const int n_live = min(per, (nq - qgrp * per * 32 + 31) >> 5);
  const int Tw = (nw + 31) >> 5;
  const int n_c = t1 - t0, n_w = z == Zn - 1 ? Tw : 0, n_it = n_c + n_w;
  const bool half_live = NW == 8 && 2 * n_live <= NW, two = half_live && n_it > FW_SHORT && tiles == 2;
  const int kg = two && wave >= n_live ? 1 : 0, wq = wave - kg * n_live;
  const bool active = wq < n_live;
  const int qt = qgrp * per + min(wq, n_live - 1), q0 = qt * 32;
  const int qi = min(q0 + c, nq - 1);
  const int r = row0 + qi / grp, head = kvh * grp + qi % grp;
  const int lo = p.row_lo[r], hi = p.row_hi[r];

  // page-table slice of this split's keys
  const int pb0 = (t0 * 32) >> ps_shift;   // page_size = 1 << ps_shift
  {
    const int pe = (min(t1 * 32, cap) + ps - 1) >> ps_shift;
    const int32_t* pt = g.page_table + (size_t)n * g.max_pages_per_seq;
    for (int i = tid; i < min(pe - pb0, pt_cap); i += T) s_pt[i] = min(max(pt[pb0 + i], 0), g.n_pages - 1);
  }

  uint4 qf[8], ql[SPLIT ? 8 : 1];
  {
    const bf16_t* qp = q + (size_t)r * q_ld + head * D + 8 * h;
#pragma unroll
    for (int ds = 0; ds < 8; ++ds) {
      qf[ds] = *(const uint4*)(qp + ds * 16);
      if (SPLIT) ql[ds] = *(const uint4*)(qp + q_lo + ds * 16);
    }
  }
  FaState st;
  st.m = -INFINITY;
  st.l = 0.f;
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) st.o[t][i] = 0.f;
  __syncthreads();   // s_pt

  // (closures capture scalars by value: captured references would pin the locals to memory)
  // Leading tiles of this split that are full tiles of cached keys (all but, at most, the last cached tile of the
  // last split).  They take forms of fetch / park / compute of their own: no clamps, no second address form, no visibility
  // mask.  A wavefront issues an instruction every four to five cycles, which is what a step of the walk waits for (its matrix
  // products and the memory take less), so the forms are chosen by branches on scalars, and with as few instructions as possible.
  const int n_fast = max(0, min(n_c, (S >> 5) - t0));
  auto tile_of = [=](int i) __attribute__((always_inline)) {
    FwTile t;
    i = min(i, n_it - 1);
    t.win = i >= n_c;
    t.kbase = (t.win ? i - n_c : t0 + i) * 32;
    t.limit = t.win ? nw : S;
    return t;
  };
  // A tile is 8 KB of keys and 8 KB of values, 16 pieces of 1 KB, a piece one load of a wavefront.  Inside a page the keys of
  // a head are contiguous, and so are its values ([D, page_size]), so a piece lies in one page: its address is the
  // page's, the piece's place in it and an offset per lane.  Piece j of the keys: rows 4 j .. + 3.  Piece j of the
  // values: kpp = min(page_size, 32) keys of page j / (kpp / 4) of the tile, for 512 / kpp head-dim rows.  Pieces 2 j and 2 j + 1 share
  // their page.
  const uint32_t pbytes = (uint32_t)Hkv * (uint32_t)ps * (D * 2);   // bytes of a page
  const int kpp_sh = min(ps_shift, 5), kpp = 1 << kpp_sh, opl = kpp_sh - 3;   // log2 of the 8-key pieces in a row
  const int vd_l = lane >> opl, vo_l = lane & ((1 << opl) - 1), vstep = (512 >> kpp_sh) * ps * 2;   // vstep: from a piece to the next of its page
  const uint64_t kb_l = (uint64_t)(k_pages + (size_t)kvh * ps * D) + lane * 16, vb_l = (uint64_t)(v_pages + (size_t)kvh * ps * D) + (vd_l * ps + vo_l * 8) * 2;
  auto v_key = [=](int j) __attribute__((always_inline)) { return (j >> (kpp_sh - 2)) * kpp; };                        // first key of piece j of the values, in its tile
  auto v_row = [=](int j) __attribute__((always_inline)) { return (j & ((kpp >> 2) - 1)) << (9 - kpp_sh); };   // and its first head-dim row
  const int kperm = fa_perm(c);
  auto compute = [=](FaState& st, const uint4 (&qf)[8], const uint4 (&ql)[SPLIT ? 8 : 1], int i, const unsigned char* buf) __attribute__((always_inline)) {
    const unsigned char* kb = buf + kperm * FW_KROW + 16 * h;
    const unsigned char* vb = buf + FW_KBUF + c * FW_VROW + 16 * h;
    f32x16_t sacc;
    S2D2_WTS(0, wave == 0 && i == 16);
#pragma unroll
    for (int j = 0; j < 16; ++j) sacc[j] = 0.f;
#pragma unroll
    for (int ds = 0; ds < 8; ++ds) {
      const uint4 kraw = *(const uint4*)(kb + ds * 32);
      if (F16) {
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, kraw), __builtin_bit_cast(f16x8_t, qf[ds]), sacc, 0, 0, 0);
      } else {
        const bf16x8_t kf = __builtin_bit_cast(bf16x8_t, kraw);
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, __builtin_bit_cast(bf16x8_t, qf[ds]), sacc, 0, 0, 0);
        if (SPLIT) sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, __builtin_bit_cast(bf16x8_t, ql[ds]), sacc, 0, 0, 0);
      }
    }
    // sacc[j]: key kbase + 16 (j / 8) + 8 h + (j % 8), query row c.  Scores stay unscaled until the exponent:
    // the running maximum is kept in scaled units, exp2(s * scale - m) is one fused multiply-add per element.
#ifdef S2D2_KERNEL_TIMING
    if (sacc[0] == 12345.678f) return;
    S2D2_WTS(1, wave == 0 && i == 16);
#endif
    float mx = -INFINITY;
    if (i < n_fast) {   // every key is visible
#pragma unroll
      for (int j = 0; j < 16; ++j) mx = fmaxf(mx, sacc[j]);
    } else {
      const FwTile t = tile_of(i);
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const int key = t.kbase + 16 * (j >> 3) + 8 * h + (j & 7);
        const int w = row0 + key;
        const int vis = (int)!t.win | ((int)(w >= lo) & (int)(w < hi)) | (int)(w == r);
        sacc[j] = ((int)(key < t.limit) & vis) ? sacc[j] : -INFINITY;
        mx = fmaxf(mx, sacc[j]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2e;
    // no divergent control flow around the MFMAs: a query row that sees nothing yet keeps m = -inf
    // and uses 0 as the reference, which makes every p below exp2(-inf) = 0
    // The reference moves only when the maximum has outgrown it by 2^8 (or there was none): the weights stay below 256, far
    // inside the half range, with the same significant bits, and the accumulators are rescaled in few tiles.
    const float m_new = mx > st.m + 8.f ? mx : st.m;
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(st.m - m_ref);
    float ls = 0.f;
    bf16x8_t pb[2], pl[SPLIT ? 2 : 1];
    f16x8_t ph16[2];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[j], scale_log2e, -m_ref));
      ls += pv;
      if (F16) {
        ph16[j >> 3][j & 7] = (_Float16)pv;
      } else {
        const __bf16 ph = (__bf16)pv;
        pb[j >> 3][j & 7] = ph;
        if (SPLIT) pl[j >> 3][j & 7] = (__bf16)(pv - (float)ph);
      }
    }
    ls += __shfl_xor(ls, 32, 64);
    st.l = st.l * alpha + ls;
    st.m = m_new;
#ifdef S2D2_KERNEL_TIMING
    if (ls == 12345.678f) return;
    S2D2_WTS(2, wave == 0 && i == 16);
#endif
    // the accumulators are rescaled only when some row's maximum moved (alpha = 1 leaves them as they are)
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int j = 0; j < 16; ++j) st.o[dt][j] *= alpha;
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint4 vraw = *(const uint4*)(vb + dt * 32 * FW_VROW + j * 32);
        if (F16) {
          st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, vraw), ph16[j], st.o[dt], 0, 0, 0);
        } else {
          const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, vraw);
          st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pb[j], st.o[dt], 0, 0, 0);
          if (SPLIT) st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pl[j], st.o[dt], 0, 0, 0);
        }
      }
    }
#ifdef S2D2_KERNEL_TIMING
    if (st.o[3][15] == 12345.678f) return;
    S2D2_WTS(3, wave == 0 && i == 16);
#endif
  };

  // Groups of KG tiles, fetched by the last FW wavefronts: one is multiplied out of one LDS buffer, the next is parked in the other one from one of
  // two register sets, which is then refilled with the group two further on; a barrier per group.
  auto walk = [&](auto kg_tag, auto fw_tag) __attribute__((always_inline)) {
    constexpr int KG = decltype(kg_tag)::value, FW = decltype(fw_tag)::value, NP = KG * 8 / FW;   // pieces of keys (and of values) per wavefront and group, all of one tile
    constexpr int PL = NP > 1 ? 2 : 1, NL = NP / PL;                // pieces per table entry, entries
    const int n_g = (n_it + KG - 1) / KG;
    if (FW < NW && wave < NW - FW) {   // the others fetch: a barrier ahead of the first tile and one behind each, as they have
      __syncthreads();
#pragma unroll 1
      for (int gi = 0; gi < n_g; ++gi) {
        if (active) compute(st, qf, ql, gi, lds + (gi & 1) * FW_BUF);
        __syncthreads();
      }
      return;
    }
    const int fwave = wave - (NW - FW), slot = fwave * NP >> 3, j0 = fwave * NP & 7;   // this wavefront's tile of a group, its first piece
    uint4 ak[NP] = {}, av[NP] = {}, bk[NP] = {}, bv[NP] = {};   // (indices are compile-time constants throughout)
    // table entries of group gi's pieces (of some valid page where there is none), read ahead of their use
    auto look = [&](int gi, uint32_t (&lk)[NL], uint32_t (&lv)[NL]) __attribute__((always_inline)) {
      const int ti = gi * KG + slot;
      const FwTile t = tile_of(ti);
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const int j = j0 + u * PL;
        lk[u] = s_pt[max(min((min(t.kbase + 4 * j, t.limit - 1) >> ps_shift) - pb0, pt_cap - 1), 0)];
        lv[u] = s_pt[max(min((min(t.kbase + v_key(j), t.limit - 1) >> ps_shift) - pb0, pt_cap - 1), 0)];
      }
    };
    auto fetch = [&](int gi, const uint32_t (&lk)[NL], const uint32_t (&lv)[NL], uint4 (&kr)[NP], uint4 (&vr)[NP]) __attribute__((always_inline)) {
      const int ti = min(gi * KG + slot, n_it - 1);   // (behind the last tile: that one again, by the code that is there already)
      if (ti < n_fast) {   // (both sides issue the same loads in the same order, so the compiler's count of those in flight holds)
        const int key = (t0 + ti) * 32;
#pragma unroll
        for (int u = 0; u < NL; ++u) {
          const int j = j0 + u * PL;
          const uint64_t ka = kb_l + ((key + 4 * j) & (ps - 1)) * (D * 2) + (uint64_t)lk[u] * pbytes;
          const uint64_t va = vb_l + (uint32_t)(((key + v_key(j)) & (ps - 1)) * 2 + v_row(j) * ps * 2) + (uint64_t)lv[u] * pbytes;
#pragma unroll
          for (int e = 0; e < PL; ++e) {
            kr[u * PL + e] = ld_kv<FW == NW>(ka + e * 1024);
            vr[u * PL + e] = ld_kv<FW == NW>(va + (uint32_t)(e * vstep));
          }
        }
      } else {
        const FwTile t = tile_of(ti);
#pragma unroll
        for (int u = 0; u < NL; ++u) {
#pragma unroll
          for (int e = 0; e < PL; ++e) {
            const int j = j0 + u * PL + e, key = t.kbase + 4 * j, keyv = t.kbase + v_key(j);
            // rows beyond the region are some rows of its last page; their scores are masked, their values zeroed in stash
            const int kc = min(key, (t.limit - 1) & ~3), kcv = min(keyv, (t.limit - 1) & ~(kpp - 1));
            const uint64_t k_c = kb_l + (kc & (ps - 1)) * (D * 2) + (uint64_t)lk[u] * pbytes;
            const uint64_t k_w = (uint64_t)(k_win + ((size_t)(row0 + min(key + (lane >> 4), nw - 1)) * Hkv + kvh) * D + (lane & 15) * 8);
            const uint64_t v_c = vb_l + (uint32_t)((kcv & (ps - 1)) * 2 + v_row(j) * ps * 2) + (uint64_t)lv[u] * pbytes;
            const uint64_t v_w = (uint64_t)(vT_win + ((size_t)(n * Hkv + kvh) * D + v_row(j) + vd_l) * wpad + min(keyv, wpad - kpp) + vo_l * 8);
            kr[u * PL + e] = ld_kv<FW == NW>(t.win ? k_w : k_c);
            vr[u * PL + e] = ld_kv<FW == NW>(t.win ? v_w : v_c);
          }
        }
      }
    };
    // half mode: cached tiles are bf16 and are converted here; the window's own rows already come as half values (k_win /
    // vT_win then point at the half copies the QKV projection wrote: 11 bits instead of the cache's 8)
    auto stash = [&](int gi, const uint4 (&kr)[NP], const uint4 (&vr)[NP]) __attribute__((always_inline)) {
      const int ti = min(gi * KG + slot, n_it - 1);
      unsigned char* buf = lds + ((gi & 1) * KG + slot) * FW_BUF;
      unsigned char* ks = buf + (4 * j0 + (lane >> 4)) * FW_KROW + (lane & 15) * 16;
      unsigned char* vs = buf + FW_KBUF + vd_l * FW_VROW + vo_l * 16;
      if (ti < n_fast) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          *(uint4*)(ks + 4 * u * FW_KROW) = F16 ? fw_to_f16(kr[u]) : kr[u];
          *(uint4*)(vs + v_row(j0 + u) * FW_VROW + v_key(j0 + u) * 2) = F16 ? fw_to_f16(vr[u]) : vr[u];
        }
      } else {
        const FwTile t = tile_of(ti);
#pragma unroll
        for (int u = 0; u < NP; ++u) {
          const uint4 vm = fw_mask(vr[u], t.limit - (t.kbase + v_key(j0 + u) + vo_l * 8));
          *(uint4*)(ks + 4 * u * FW_KROW) = F16 && !t.win ? fw_to_f16(kr[u]) : kr[u];
          *(uint4*)(vs + v_row(j0 + u) * FW_VROW + v_key(j0 + u) * 2) = F16 && !t.win ? fw_to_f16(vm) : vm;
        }
      }
    };
    auto pass = [&](int gi, uint4 (&kr)[NP], uint4 (&vr)[NP]) __attribute__((always_inline)) {
      uint32_t lk[NL], lv[NL];
      look(gi + 3, lk, lv);
      if (FW == NW && active && gi >= 0 && gi * KG + kg < n_it) compute(st, qf, ql, gi * KG + kg, lds + ((gi & 1) * KG + kg) * FW_BUF);
      if (gi + 1 >= 0 && gi + 1 < n_g) stash(gi + 1, kr, vr);
      fetch(gi + 3, lk, lv, kr, vr);
      if (gi >= -1) __syncthreads();
    };
    // (gi < 0: the first groups' loads, nothing to multiply yet.  One copy of the pass per register set: most launches over
    // short caches are four tiles a workgroup, and instructions that are executed once come from memory.)
#pragma unroll 1
    for (int gi = -3;; gi += 2) {
      pass(gi, ak, av);
      if (gi + 1 >= n_g) break;
      pass(gi + 1, bk, bv);
      if (gi + 2 >= n_g) break;
    }
  };
  // Four wavefronts (two workgroups to a compute unit): one tile at a time, every thread fetches two pieces of keys and of
  // values (K row idx / 16, 16-byte piece idx % 16; V^T row idx / 4, keys 8 (idx % 4) .. + 8), one tile in flight, in forms
  // compiled for full cached tiles (FAST) and for all.  Walked two tiles at a time like eight wavefronts, launches of short splits
  // took 1 to 4 us longer (1.7B shape, four tiles a split, with the merge 25 for 19) and long ones were as fast.
  auto walk4 = [&](auto stream_tag) __attribute__((always_inline)) {
    constexpr bool STREAM = decltype(stream_tag)::value;
    constexpr std::true_type FT_{};
    constexpr std::false_type GT_{};
    const size_t pstride = (size_t)Hkv * ps * D;   // elements of a page
    auto fetch1 = [=](auto fast, int u, int i, uint4& kr, uint4& vr) __attribute__((always_inline)) {
      constexpr bool FAST = decltype(fast)::value;
      const int idx = tid + u * T, kk = idx >> 4, kch = idx & 15, vd = idx >> 2, vko = (idx & 3) * 8;
      // (offsets are page * page_stride + [terms that depend on the thread alone] + [32-bit terms of the tile])
      if (FAST) {
        const int key = (t0 + i) * 32 + kk, kv0 = (t0 + i) * 32 + vko;
        const int pk = s_pt[min((key >> ps_shift) - pb0, pt_cap - 1)];
        const int pv = s_pt[min((kv0 >> ps_shift) - pb0, pt_cap - 1)];
        kr = ld_kv<STREAM>((uint64_t)(k_pages + ((size_t)kvh * ps * D + kch * 8) + (size_t)pk * pstride + (key & (ps - 1)) * D));
        vr = ld_kv<STREAM>((uint64_t)(v_pages + ((size_t)kvh * D + vd) * ps + (size_t)pv * pstride + (kv0 & (ps - 1))));
        return;
      }
      const FwTile t = tile_of(i);
      const int key = min(t.kbase + kk, t.limit - 1);   // rows beyond the region read a valid row; their scores are masked
      const int key0 = t.kbase + vko;
      // both address forms are computed and one is selected: no control flow around the loads
      const int kv0 = min(key0, cap - 8);
      const int pk = s_pt[max(0, min((key >> ps_shift) - pb0, pt_cap - 1))];
      const int pv = s_pt[max(0, min((kv0 >> ps_shift) - pb0, pt_cap - 1))];
      const bf16_t* kp_c = k_pages + ((size_t)kvh * ps * D + kch * 8) + (size_t)pk * pstride + (key & (ps - 1)) * D;
      const bf16_t* vp_c = v_pages + ((size_t)kvh * D + vd) * ps + (size_t)pv * pstride + (kv0 & (ps - 1));
      const bf16_t* kp_w = k_win + ((size_t)row0 * Hkv + kvh) * D + kch * 8 + (size_t)key * (Hkv * D);
      const bf16_t* vp_w = vT_win + ((size_t)(n * Hkv + kvh) * D + vd) * wpad + min(key0, wpad - 8);
      kr = ld_kv<STREAM>((uint64_t)(t.win ? kp_w : kp_c));
      vr = ld_kv<STREAM>((uint64_t)(t.win ? vp_w : vp_c));
    };
    auto stash1 = [=](auto fast, int u, int i, int b, uint4 kr, uint4 vr) __attribute__((always_inline)) {
      constexpr bool FAST = decltype(fast)::value;
      unsigned char* base = lds + b * FW_BUF;
      const int idx = tid + u * T, kk = idx >> 4, kch = idx & 15, vd = idx >> 2, vko = (idx & 3) * 8;
      const FwTile t = FAST ? FwTile{false, 0, 0} : tile_of(i);
      const uint4 vm = FAST || t.kbase + 32 <= t.limit ? vr : fw_mask(vr, t.limit - (t.kbase + vko));   // (uniform: only a region's last tile is partial)
      const bool cvt = F16 && (FAST || !t.win);
      *(uint4*)(base + kk * FW_KROW + kch * 16) = cvt ? fw_to_f16(kr) : kr;
      *(uint4*)(base + FW_KBUF + vd * FW_VROW + vko * 2) = cvt ? fw_to_f16(vm) : vm;
    };
    uint4 k0, v0, k1, v1;
    fetch1(GT_, 0, 0, k0, v0);
    fetch1(GT_, 1, 0, k1, v1);
    stash1(GT_, 0, 0, 0, k0, v0);
    stash1(GT_, 1, 0, 0, k1, v1);
    fetch1(GT_, 0, 1, k0, v0);
    fetch1(GT_, 1, 1, k1, v1);
    __syncthreads();
    // one pass: computes tile i, parks tile i + 1, requests tile i + 2
    auto pass = [&](auto fast, int i) __attribute__((always_inline)) {
      if (active) compute(st, qf, ql, i, lds + (i & 1) * FW_BUF);
      stash1(fast, 0, i + 1, (i + 1) & 1, k0, v0);
      stash1(fast, 1, i + 1, (i + 1) & 1, k1, v1);
      fetch1(fast, 0, i + 2, k0, v0);
      fetch1(fast, 1, i + 2, k1, v1);
      __syncthreads();
    };
    int i = 0;
    for (; i + 2 < n_fast; ++i) pass(FT_, i);
    for (; i < n_it; ++i) pass(GT_, i);
  };
  if (n_it > 0) {
    if constexpr (NW == 4) {
      if (n_it > FW_SHORT4 || n_splits * (int)gridDim.x <= cus) walk4(std::true_type{});
      else walk4(std::false_type{});
    }
    else if (two) walk(std::integral_constant<int, 2>{}, std::integral_constant<int, NW>{});
    else if (half_live) walk(std::integral_constant<int, 1>{}, std::integral_constant<int, NW / 2>{});
    else walk(std::integral_constant<int, 1>{}, std::integral_constant<int, NW>{});
  }
  if (NW == 8 && two) {   // the second key group's states, through LDS (behind the last group's barrier: nobody reads tiles any more)
    float4* s_o = (float4*)lds;                                    // [query tile][16][lane]
    float2* s_ml = (float2*)(lds + (NW / 2) * 16384);              // [query tile][lane]
    if (kg == 1 && active) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          s_o[(wq * 16 + dt * 4 + i4) * 64 + lane] = make_float4(st.o[dt][4 * i4], st.o[dt][4 * i4 + 1], st.o[dt][4 * i4 + 2], st.o[dt][4 * i4 + 3]);
      s_ml[wq * 64 + lane] = make_float2(st.m, st.l);
    }
    __syncthreads();
    if (kg == 1 || !active) return;
    const float2 ml = s_ml[wq * 64 + lane];
    const float M = fmaxf(st.m, ml.x), ref = M == -INFINITY ? 0.f : M;
    const float f0 = __builtin_amdgcn_exp2f(st.m - ref), f1 = __builtin_amdgcn_exp2f(ml.x - ref);
    st.m = M;
    st.l = st.l * f0 + ml.y * f1;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const float4 v = s_o[(wq * 16 + dt * 4 + i4) * 64 + lane];
        st.o[dt][4 * i4] = st.o[dt][4 * i4] * f0 + v.x * f1;
        st.o[dt][4 * i4 + 1] = st.o[dt][4 * i4 + 1] * f0 + v.y * f1;
        st.o[dt][4 * i4 + 2] = st.o[dt][4 * i4 + 2] * f0 + v.z * f1;
        st.o[dt][4 * i4 + 3] = st.o[dt][4 * i4 + 3] * f0 + v.w * f1;
      }
  }

  // ---- output: lane (c, h) holds head-dim positions dt*32 + 8*i4 + 4*h .. + 4 of query row c ----
  const size_t item0 = ((size_t)item * q_tiles + qt) * Z;
  if (Zn == 1) {
    if (active && q0 + c < nq) {
      const float inv = st.l > 0.f ? 1.0f / st.l : 0.f;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
          fa_store4<false>(o, o_lo, r, head * D + 4 * h + dt * 32 + 8 * i4, o_ld, st.o[dt][4 * i4] * inv, st.o[dt][4 * i4 + 1] * inv,
                           st.o[dt][4 * i4 + 2] * inv, st.o[dt][4 * i4 + 3] * inv);
    }
    return;
  }
  // the splits' partials, in register order; attn_wide_merge_kernel, launched next, adds them up
  if (active) {
    float* po = part_o + (item0 + z) * 32 * D + (size_t)lane * 4;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        *(float4*)(po + (dt * 4 + i4) * 256) = make_float4(st.o[dt][4 * i4], st.o[dt][4 * i4 + 1], st.o[dt][4 * i4 + 2], st.o[dt][4 * i4 + 3]);
    if (h == 0) {
      part_ml[(item0 + z) * 64 + c] = st.m;
      part_ml[(item0 + z) * 64 + 32 + c] = st.l;
    }
  }
}

// Sums of the key splits, in split order: one wavefront per 32 query rows x 8 output columns (the 64 x 16 bytes its
// accumulator group has in every split), the partials of all splits up to 12 requested at once (always of 12, with the last one again
// where there are fewer: 9.0 -> 6.8 us per launch for two splits of 32 sequences).  A launch of its own costs 5-7 us of
// latency, 7-11 where it reads tens of MB of partials (8B and MoE); when the split that arrived last added up its
// workgroup's tiles by itself, that was one memory round trip per query tile, pass and four splits behind each other, on one
// compute unit, 6 to 27 us of the launch.  Attention and merge per launch before and now: 4B verifier 46 -> 28 + 6 us (with
// equal runs of tiles per split), 8B verifier 166 -> 142 + 12, 8B draft 126 -> 114 + 9, MoE draft 79 -> 48 + 14 (the merges with
// loads of 12 splits).
__global__ __launch_bounds__(256) void attn_wide_merge_kernel(const float* __restrict__ part_o, const float* __restrict__ part_ml, KvGeom g,
                                                              Plan p, int Hq, int Z, bf16_t* __restrict__ o, int o_ld, int o_lo) {
  constexpr int D = FA_D;
  const int lane = threadIdx.x & 63, g16 = blockIdx.x * 4 + (threadIdx.x >> 6), qt = blockIdx.y, item = blockIdx.z;
  const int Hkv = g.n_kv_heads, grp = Hq / Hkv, n = item / Hkv, kvh = item % Hkv, c = lane & 31;
  const int row0 = p.seq_row0[n], nq = p.seq_rows[n] * grp, Zn = p.seq_splits[n];
  if (Zn == 1 || qt * 32 >= nq) return;
  const size_t item0 = ((size_t)item * gridDim.y + qt) * Z;
  float M = -INFINITY, L = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto rounds = [&](auto zb) __attribute__((always_inline)) {
    constexpr int ZB = decltype(zb)::value;
    for (int z0 = 0; z0 < Zn; z0 += ZB) {
      float m[ZB], l[ZB];
      float4 v[ZB];
#pragma unroll
      for (int k = 0; k < ZB; ++k) {
        const size_t e = item0 + min(z0 + k, Zn - 1);   // clamped duplicates get no weight below
        m[k] = part_ml[e * 64 + c];
        l[k] = part_ml[e * 64 + 32 + c];
        v[k] = *(const float4*)(part_o + e * 32 * D + (g16 * 64 + lane) * 4);
      }
      float Mn = M;
#pragma unroll
      for (int k = 0; k < ZB; ++k) {
        if (z0 + k >= Zn) m[k] = -INFINITY;
        Mn = fmaxf(Mn, m[k]);
      }
      const float ref = Mn == -INFINITY ? 0.f : Mn;   // (nothing seen yet: all weights are exp2(-inf) = 0)
      const float fo = __builtin_amdgcn_exp2f(M - ref);
      L *= fo; acc.x *= fo; acc.y *= fo; acc.z *= fo; acc.w *= fo;
#pragma unroll
      for (int k = 0; k < ZB; ++k) {
        const float f = __builtin_amdgcn_exp2f(m[k] - ref);
        L += f * l[k];
        acc.x += f * v[k].x; acc.y += f * v[k].y; acc.z += f * v[k].z; acc.w += f * v[k].w;
      }
      M = Mn;
    }
  };
  if (Zn <= 2) rounds(std::integral_constant<int, 2>{});
  else if (Zn <= 4) rounds(std::integral_constant<int, 4>{});
  else if (Zn <= 8) rounds(std::integral_constant<int, 8>{});
  else rounds(std::integral_constant<int, 12>{});
  const int qi = qt * 32 + c, d0 = (g16 >> 2) * 32 + 8 * (g16 & 3) + 4 * (lane >> 5);
  if (qi >= nq) return;
  const float inv = L > 0.f ? 1.0f / L : 0.f;
  fa_store4<false>(o, o_lo, row0 + qi / grp, (kvh * grp + qi % grp) * D + d0, o_ld, acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
}

template <int NW>
static void launch_wide(hipStream_t st, int qm, dim3 grid, size_t lds, const bf16_t* q, int q_ld, int q_lo,
                        const bf16_t* k_win, const bf16_t* vT_win, const bf16_t* kp, const bf16_t* vp, const KvGeom& g,
                        const Plan& p, int Hq, int Z, int wpad, float scale_log2e, bf16_t* o, int o_ld, int o_lo,
                        float* part_o, float* part_ml, int q_tiles, int per, int pt_cap, int ps_shift, int tiles, int cus) {
#define S2D2_WIDE_QM(QMV)                                                                                                    \
  S2D2_LAUNCH((attn_flash_wide_kernel<NW, QMV>), grid, dim3(NW * 64), lds, st, q, q_ld, q_lo, k_win, vT_win, kp, vp, g, p, \
              Hq, Z, wpad, scale_log2e, o, o_ld, o_lo, part_o, part_ml, q_tiles, per, pt_cap, ps_shift, tiles, cus)
  if (qm == OPM_F16) S2D2_WIDE_QM(OPM_F16);
  else if (qm == OPM_BF16X2) S2D2_WIDE_QM(OPM_BF16X2);
  else S2D2_WIDE_QM(OPM_BF16);
#undef S2D2_WIDE_QM
}

// Query tiles of a workgroup, of q_tiles that there is room for and `expected` ones that have rows.  Up to five expected: one workgroup for up to
// eight tiles, so that a tile of keys is fetched once (where at most four have rows its eight wavefronts stand in two key groups).  More: up to four
// tiles, as many in every workgroup that has rows: cut by the room, half as much again for a verifier, one
// workgroup had all rows but those of a tile or two.  Forwards, us, by the room in eights / expected in fours / expected in eights: 8B verification
// of 16 sequences behind 2000 to 4000, 5 expected of 8 15317 / 15419 / 17404, 6 of 9 18923 / 16695 / 18751, 7 of 11 21599 / 20342 / 21436, 8 of 12 22561 / 21358 /
// 22477; 4B 3 sequences 6 of 8 4566 / 4480 / 4478, 4 sequences 7 of 11 5488 / 5413 / 5468; MoE 6 sequences 8 of 12 5046 / 4991 / 5080; 1.7B prefill 12 of 12 15964 / 15723
// / 15929.
int attention_wide_per(int q_tiles, int expected) {
  const int most = expected > 5 ? 4 : 8, over = expected > 5 ? expected : q_tiles, groups = (over + most - 1) / most;
  return (over + groups - 1) / groups;
}

// Wavefronts of a workgroup: eight for more than four tiles, and for up to four where sequences, heads and groups are at most 128 workgroups ahead of the
// key splits: four multiply every other tile each, or four fetch.  With more of them a launch has few splits to even out ragged caches with, and twice as
// many workgroups of four are worth more.  (Two wavefronts for two tiles: slower, four share the fetch work.)  Forwards, us, four / eight wavefronts:
// workgroups 40 1.7B verification in mid-block 1821 / 1717, 48 4B 6 tiles 4551 / 4351, 64 4B verification 4816 / 4732, 96 1.7B prefill 15824 / 15399, 96 4B draft behind
// 4000 to 8000 5588 / 5510, 128 8B draft behind 8192 10777 / 10537, MoE verification 5232 / 5186, 192 8B draft behind 500 to 3000 8736 / 8932, 256 4B draft
// 7064 / 7116, 8B verification of 6 tiles 16847 / 17866.
int attention_wide_nw(int per, int wgs) { return per > 4 || wgs <= 128 ? 8 : 4; }

// Most splits of a sequence: a split keeps at least four key tiles, the partials fit their buffer.  One, and so no merge
// launch, where the cache holds so few tiles that cutting them saves less than that launch costs (2-3 us when nothing was
// cut, 5-11 else), which depends on how many workgroups there are without: forwards over prefixes that fill their cache,
// uncut against cut, us: 32 sequences of block 8, 4B (256 workgroups) 6 tiles 6460 / 6700, 8 6614 / 6795, 10 6666 / 6916, 13
// 6740 / 6846; 21 sequences, two planes (168) 6 tiles 7800 / 7943, 8 7916 / 8039, 10 7972 / 7999, 13 8153 / 8082; 16
// sequences (128) 6 tiles 4762 / 4823, 8 4868 / 4839; one sequence (8) 6 tiles 1593 / 1574.
int attention_wide_splits(const KvGeom& g, int items, int q_tiles, int groups, size_t part_entries, int target) {
  const int cap_tiles = (g.max_pages_per_seq * g.page_size + 31) / 32, wgs = items * groups;
  if (cap_tiles <= (wgs >= 256 ? 18 : wgs >= 128 ? 7 : WIDE_MIN_TILES)) return 1;
  int Z = std::max(1, std::min(std::min((cap_tiles + WIDE_MIN_TILES - 1) / WIDE_MIN_TILES, 64), target + 1));
  while (Z > 1 && (size_t)Z * items * q_tiles > part_entries) --Z;
  return Z;
}

// Tiles of a split at most: N sequences of the cache's capacity share the target's splits, a single one has at most Z.
int attention_wide_run_most(const KvGeom& g, int N, int Z, int target) {
  const int cap_tiles = (g.max_pages_per_seq * g.page_size + 31) / 32;
  return (int)std::max((long long)std::max((cap_tiles + Z - 1) / Z, WIDE_MIN_TILES), ((long long)N * cap_tiles + target - 1) / target);
}
// Page-table entries a split can touch (plus slack for the ragged ends).
int attention_wide_pt_cap(const KvGeom& g, int N, int Z, int target) {
  return (int)std::min((long long)g.max_pages_per_seq, ((long long)attention_wide_run_most(g, N, Z, target) + 1) * 32 / g.page_size + 2);
}

void launch_attention_wide(hipStream_t st, const void* q, int q_ld, int q_lo, const void* k_win, const void* vT_win,
                           const void* k_pages_layer, const void* v_pages_layer, const KvGeom& g, const Plan& p, int N,
                           int Hq, int q_tiles, int per, int nw, int Z, int target, int tiles, int cus, int wpad, void* o, int o_ld, int o_lo, float* part,
                           size_t part_entries) {
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)g.head_dim);
  const int qgroups = (q_tiles + per - 1) / per;
  const int pt_cap = attention_wide_pt_cap(g, N, Z, target);
  float* part_o = part;
  float* part_ml = part + part_entries * 32 * FA_D;
  const dim3 grid(g.n_kv_heads, qgroups, std::min(N * Z, N + target));   // (N + target: a run more than the target per sequence at most)
  const size_t lds = attention_wide_lds_bytes(pt_cap, tiles);
  int ps_shift = 0;
  while ((1 << ps_shift) < g.page_size) ++ps_shift;   // the caller has checked that page_size is a power of two
#define S2D2_WIDE(NWV)                                                                                                  \
  launch_wide<NWV>(st, operand_mode(q_lo), grid, lds, (const bf16_t*)q, q_ld, q_lo, (const bf16_t*)k_win, (const bf16_t*)vT_win, \
                   (const bf16_t*)k_pages_layer, (const bf16_t*)v_pages_layer, g, p, Hq, Z, wpad, scale_log2e,          \
                   (bf16_t*)o, o_ld, o_lo, part_o, part_ml, q_tiles, per, pt_cap, ps_shift, tiles, cus)
  if (nw == 4) S2D2_WIDE(4);
  else S2D2_WIDE(8);
#undef S2D2_WIDE
}

void launch_attention_wide_merge(hipStream_t st, const KvGeom& g, const Plan& p, int N, int Hq, int q_tiles, int Z, void* o, int o_ld,
                                 int o_lo, const float* part, size_t part_entries) {
  S2D2_LAUNCH(attn_wide_merge_kernel, dim3(4, q_tiles, N * g.n_kv_heads), dim3(256), 0, st, part, part + part_entries * 32 * FA_D, g, p, Hq, Z,
              (bf16_t*)o, o_ld, o_lo);
}

template <int NW, int QM>
static hipError_t wide_lds_limit() {
  return hipFuncSetAttribute((const void*)attn_flash_wide_kernel<NW, QM>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
}

int attention_wide_init() {
  hipError_t e = hipSuccess;
#define S2D2_LIM(NWV)                                                          \
  if (e == hipSuccess) e = wide_lds_limit<NWV, OPM_BF16>();                    \
  if (e == hipSuccess) e = wide_lds_limit<NWV, OPM_BF16X2>();                  \
  if (e == hipSuccess) e = wide_lds_limit<NWV, OPM_F16>();
  S2D2_LIM(4) S2D2_LIM(8)
#undef S2D2_LIM
  return e == hipSuccess ? 0 : -1;
}

}  // namespace s2d2
