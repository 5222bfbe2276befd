// GEMM on the packed weights for windows between the streaming kernel's 16 rows and the blocks of gemm_block.hip:
//   Y[m, n] = sum_k X[m, k] W[n, k],  17 to 48 rows (unembedding of small vocabularies: 64), half operands, X in fragment order (LO_F16P).
//
// At these sizes a launch is bound by reading the weights once, and on the way there by everything that is not the
// K loop: the tiled kernel pads the rows to 128, splits K over compute units to fill the chip, and pays row maps,
// a 64-128 KB partial per workgroup and its merge (20-35 us per launch whatever the matrix).  Here, as in the streaming
// kernel, every operand goes straight from memory to a matrix instruction: a weight fragment is multiplied with RB
// activation fragments, all of them 1 KB of contiguous memory.  No LDS and no barrier in the K loop; the eight
// wavefronts of a workgroup split K, their sums meet in LDS in wavefront order, and every wavefront finishes its share
// of the 16 x 16 units.
//
// What bounds it: the weights come from memory at 6.6 TB/s at best (reads alone), the activation fragments from L2 at
// about 20 TB/s, and the two do not overlap (measured on a copy of the load pattern: with TA weight and RB activation
// fragments per K tile a launch takes W / 6.7 + X / 27 TB/s, whatever is in flight beyond two tiles per wavefront).  The
// activations are read once per workgroup, so a workgroup takes as many feature tiles as the accumulators allow
// (TA = 1 .. 6), one workgroup of 256 registers per compute unit, and where the groups of tiles do not fill the chip
// K is also shared by KS workgroups.  Measured (4B-shaped layer, 64 rows, us per launch): QKV 13.5, output 12.9, gate / up
// 27.3 (100 MB: 3.7 TB/s), down 18.9; the tiled kernel took 25.5, 22.9, 35.4, 32.6.
//
// The row count is on the device: the weights of the first tiles are requested before it is known, then the kernel
// switches on the row blocks there are (compiled for 1 .. 4 of them); more rows than 64 are taken by further workgroups.
#include "gemm_epilogue.h"
#include "../../include/s2d2.h"

#include <algorithm>

namespace s2d2 {

static constexpr int MID_NW = 8, MID_RB = 4;   // wavefronts; most row blocks of 16 of a workgroup

// LDS accesses of this wavefront done, then the workgroup's barrier; global loads stay in flight.
__device__ __forceinline__ void mid_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Rows m0 .. of the window (at most 16 RB of them); w holds the first U tiles of the workgroup's first group.
template <int EPI, int TPW, int RB, int U, bool SHARED>
__device__ __forceinline__ void gemm_mid_body(const GemmStreamArgs& a, u32x4_t (&w)[TPW * (EPI == SEPI_SWIGLU ? 2 : 1)][U],
                                              const int m0, const int M, const int KS_, uint8_t* smem) {
  constexpr int NACC = EPI == SEPI_SWIGLU ? 2 : 1, TA = TPW * NACC, NU = RB * TPW, HW = MID_NW / 2;
  const int KS = SHARED ? KS_ : 1;
  // (opaque: what depends on the thread index alone is otherwise computed ahead of the switch for all row counts and spilled)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (scalar: K bounds must give scalar branches)
  const int g = lane >> 4, f = lane & 15;
  const int Mloc = min(RB * 16, M - m0), KT = a.KT, groups = (a.NT + TPW - 1) / TPW;
  const int sets = gridDim.x / KS, ks = KS - 1 - (int)blockIdx.x / sets, set = blockIdx.x % sets;
  const int share = ks * MID_NW + wave, kb = share * (KT / U) / (MID_NW * KS) * U, ke = (share + 1) * (KT / U) / (MID_NW * KS) * U;
  float* s_rs = (float*)smem;                       // [128] 1/rms of the rows
  f32x4_t* s_red = (f32x4_t*)(smem + 512);          // [wavefront of a half][unit][accumulator][lane]

  // Every load is 64 lanes x 16 contiguous bytes: scalar tile address + 16 lane (gathered rows: + an offset per lane).
  const int32_t* gather = EPI == SEPI_STORE_F32 ? a.gather : nullptr;
  uint32_t xo[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r0 = m0 + min(rb * 16, (Mloc - 1) & ~15);   // blocks past the rows read the last one again; never stored
    if (EPI == SEPI_STORE_F32) xo[rb] = 2u * (uint32_t)(gather ? frag_offset(gather[min(r0 + f, M - 1)], 8 * g, a.K) : frag_offset(r0 + f, 8 * g, a.K));
    else xo[rb] = (uint32_t)(r0 >> 4) * (uint32_t)KT * 1024u;
  }
  const uint32_t lane16 = lane * 16;
  u32x4_t x[RB][U];
  const u32x4_t* wp[TA];   // the group's weight tiles, K tile 0
  auto point = [&](int grp) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const size_t at = (size_t)min(grp * TPW + t, a.NT - 1) * KT * 64;
      wp[t * NACC] = (const u32x4_t*)a.Wp + at;
      if (NACC == 2) wp[t * NACC + 1] = (const u32x4_t*)a.Wp2 + at;
    }
  };
  auto load_w = [&](int u, int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TA; ++t) w[t][u] = ld_stream((const u32x4_t*)((const uint8_t*)(wp[t] + (size_t)kt * 64) + lane16));
  };
  auto load_x = [&](int u, int kt) __attribute__((always_inline)) {
    const uint8_t* xk = (const uint8_t*)a.X + (size_t)kt * 1024;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) x[rb][u] = EPI == SEPI_STORE_F32 ? *(const u32x4_t*)(xk + xo[rb]) : *(const u32x4_t*)(xk + xo[rb] + lane16);
  };
  int grp = set;
  point(grp);
#pragma unroll
  for (int u = 0; u < U; ++u) load_x(u, kb + u);
  __builtin_amdgcn_sched_barrier(0);

  // ---- 1/rms of the rows from the producer's partial sums of squares, behind the first tiles (the accumulators'
  // registers are still free) ----
  if (EPI != SEPI_ADD_F32) {
    constexpr int TPR = RB == 1 ? 32 : RB == 2 ? 16 : 8;   // threads per row
    constexpr int SSV = 64 / TPR;                           // float4 per thread and round
    const int ss_row = tid / TPR, ss_sub = tid % TPR;
    const int rr = min(m0 + ss_row, M - 1);   // rows past the count read a valid row; their 1/rms is never used
    const float* pp = a.ss_part + (size_t)(gather ? gather[rr] : rr) * a.ss_stride;
    float v = 0.f;
    if ((a.ss_count & 3) == 0 && (a.ss_stride & 3) == 0) {
      const int n4 = a.ss_count >> 2;
      for (int i0 = ss_sub; i0 < n4; i0 += TPR * SSV) {
        float4 t[SSV];
#pragma unroll
        for (int j = 0; j < SSV; ++j) t[j] = ((const float4*)pp)[min(i0 + TPR * j, n4 - 1)];   // clamped duplicates are skipped when summing
#pragma unroll
        for (int j = 0; j < SSV; ++j)
          if (i0 + TPR * j < n4) v += (t[j].x + t[j].y) + (t[j].z + t[j].w);
      }
    } else {
      for (int i = ss_sub; i < a.ss_count; i += TPR) v += pp[i];
    }
#pragma unroll
    for (int off = 1; off < TPR; off <<= 1) v += __shfl_xor(v, off, 64);
    if (ss_row < RB * 16 && ss_sub == 0) s_rs[ss_row] = 1.0f / sqrtf(v / (float)a.K + a.eps);
  }

  for (bool more = true; more;) {
    f32x4_t acc[RB][TA];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int t = 0; t < TA; ++t) acc[rb][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mac = [&](int u) __attribute__((always_inline)) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < TA; ++t) acc[rb][t] = mfma_16x16x32<OPM_F16>(w[t][u], x[rb][u], acc[rb][t]);
    };
    // sliding window over the K tiles: a slot is refilled right after its last use (see the streaming kernel)
    // (shares are whole batches of U tiles, at least one: a condition on single tiles would keep a second copy of the
    // accumulators)
    for (int kt0 = kb + U; kt0 < ke; kt0 += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        mac(u);
        load_w(u, kt0 + u);
        load_x(u, kt0 + u);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) mac(u);
    const int cgrp = grp;
    grp += sets;
    more = !SHARED && grp < groups;

    // ---- the wavefronts' sums, through LDS: the upper four add theirs to the lower four's, then every wavefront sums
    // its units (wave, wave + 8, ...) over the four.  The residual values a unit is added to are requested ahead of
    // that, and behind them the first tiles of the next group. ----
    int lm = lane;   // (opaque again: the addresses of the merge are not to be kept in registers across the K loop)
    asm volatile("" : "+v"(lm));
    const int gm = lm >> 4, fm = lm & 15;
    mid_barrier();   // (the group before has been read)
    if (wave >= HW) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < TA; ++t) s_red[(((wave - HW) * RB + rb) * TA + t) * 64 + lm] = acc[rb][t];
    }
    mid_barrier();
    if (wave < HW) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < TA; ++t) {
          f32x4_t* p = &s_red[((wave * RB + rb) * TA + t) * 64 + lm];
          *p = acc[rb][t] + *p;
        }
    }
    constexpr int UPW = (NU + MID_NW - 1) / MID_NW;
    float4 h0[UPW];
#pragma unroll
    for (int q = 0; q < UPW; ++q) {
      h0[q] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (EPI == SEPI_ADD_F32) {
        const int u = min(wave + MID_NW * q, NU - 1), r = min(m0 + (u / TPW) * 16 + fm, M - 1), nt = min(cgrp * TPW + u % TPW, a.NT - 1);
        h0[q] = *(const float4*)((const float*)a.out + (size_t)r * a.ldo + nt * 16 + 4 * gm);
      }
    }
    if (more) {
      point(grp);
#pragma unroll
      for (int u = 0; u < U; ++u) { load_w(u, kb + u); load_x(u, kb + u); }
    }
    mid_barrier();
#pragma unroll
    for (int q = 0; q < UPW; ++q) {
      const int u = wave + MID_NW * q;
      if (u >= NU) break;
      const int rb = u / TPW, t = u % TPW, nt = cgrp * TPW + t;
      if (rb * 16 >= Mloc || nt >= a.NT) continue;   // uniform over the wavefront
      f32x4_t sum[NACC];
#pragma unroll
      for (int c = 0; c < NACC; ++c) {
        f32x4_t p[HW];
#pragma unroll
        for (int wv = 0; wv < HW; ++wv) p[wv] = s_red[((wv * RB + rb) * TA + t * NACC + c) * 64 + lm];
        sum[c] = (p[0] + p[1]) + (p[2] + p[3]);
      }
      if (SHARED) {
        // K shared by KS workgroups (one group each): the shares 1 .. KS - 1 (first in dispatch order; they never wait) hand
        // their sums over as 64-bit (value, tag) words; share 0 requests the words of all of them at once until all
        // are there, adds them in share order, clears them for the next launch and finishes the unit.  The
        // wait is bounded; one that runs out sets *pair_status and goes on with what is there.
        constexpr int KSM = 4;
        unsigned long long* slot0 = a.pair_buf + (((size_t)blockIdx.y * sets + set) * (KSM - 1) * MID_RB * TA + u * NACC) * 256 + lm;
        if (ks > 0) {
          unsigned long long* slot = slot0 + (size_t)(ks - 1) * MID_RB * TA * 256;
#pragma unroll
          for (int c = 0; c < NACC; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              __hip_atomic_store(slot + c * 256 + i * 64, (unsigned long long)__float_as_uint(sum[c][i]) | (1ull << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          continue;
        }
        unsigned long long v[KSM - 1][NACC][4];
        int spins = 0;
        for (; spins < (1 << 20); ++spins) {
          unsigned long long all = ~0ull;
#pragma unroll
          for (int k = 0; k < KSM - 1; ++k) {
            const size_t ko = (size_t)min(k, KS - 2) * MID_RB * TA * 256;   // (fewer shares: the last one again)
#pragma unroll
            for (int c = 0; c < NACC; ++c)
#pragma unroll
              for (int i = 0; i < 4; ++i) v[k][c][i] = __hip_atomic_load(slot0 + ko + c * 256 + i * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
#pragma unroll
          for (int k = 0; k < KSM - 1; ++k)
#pragma unroll
            for (int c = 0; c < NACC; ++c)
#pragma unroll
              for (int i = 0; i < 4; ++i) all &= v[k][c][i];
          if (all >> 32) break;
        }
        if (spins == (1 << 20) && a.pair_status) *a.pair_status = 1;
#pragma unroll
        for (int k = 0; k < KSM - 1; ++k) {
          if (k >= KS - 1) break;   // uniform
#pragma unroll
          for (int c = 0; c < NACC; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              __hip_atomic_store(slot0 + (size_t)k * MID_RB * TA * 256 + c * 256 + i * 64, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              sum[c][i] += __uint_as_float((uint32_t)v[k][c][i]);
            }
        }
      }
      const int r = rb * 16 + fm;
      gemm_epi_unit<EPI, true>(a, r < Mloc, m0 + min(r, Mloc - 1), EPI == SEPI_ADD_F32 ? 1.0f : s_rs[r], nt, gm, sum[0], sum[NACC - 1], &h0[q]);
    }
  }
}

// Tiles in flight per wavefront (U): what fits next to the accumulators in 256 registers.
constexpr int mid_u(int TA) {
  return 4 * MID_RB * TA + 16 * (MID_RB + TA) <= 150 ? 4 : 2;
}

template <int EPI, int TPW, bool SHARED>
__global__ __launch_bounds__(MID_NW * 64, 2) void gemm_mid_kernel(const GemmStreamArgs a, const int KS_) {
  extern __shared__ __align__(16) uint8_t smem[];
  constexpr int NACC = EPI == SEPI_SWIGLU ? 2 : 1, TA = TPW * NACC, U = mid_u(TA);
  const int KS = SHARED ? KS_ : 1;
  const int m0 = blockIdx.y * 16 * MID_RB;
  int M = 0;
  if (blockIdx.y != 0) {   // passes the row count may not need: request no weights for nothing
    M = *a.m_count;
    if (m0 >= M) return;
  }
  u32x4_t w[TA][U];
  {   // the weights of the first tiles: their addresses need no row count
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), KT = a.KT;
    const int sets = gridDim.x / KS, ks = KS - 1 - (int)blockIdx.x / sets, set = blockIdx.x % sets;
    const int share = ks * MID_NW + wave, kb = share * (KT / U) / (MID_NW * KS) * U;
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const size_t at = ((size_t)min(set * TPW + t, a.NT - 1) * KT + kb + u) * 64;
        w[t * NACC][u] = ld_stream((const u32x4_t*)((const uint8_t*)((const u32x4_t*)a.Wp + at) + (uint32_t)lane * 16));
        if (NACC == 2) w[t * NACC + 1][u] = ld_stream((const u32x4_t*)((const uint8_t*)((const u32x4_t*)a.Wp2 + at) + (uint32_t)lane * 16));
      }
    }
  }
  if (blockIdx.y == 0) M = *a.m_count;
  if (M <= m0) return;
  const int nb = min(MID_RB, (M - m0 + 15) >> 4);
#define S2D2_MID_BODY(RB) gemm_mid_body<EPI, TPW, RB, U, SHARED>(a, w, m0, M, KS, smem)
  if (nb == 1) S2D2_MID_BODY(1);
  else if (nb == 2) S2D2_MID_BODY(2);
  else if (nb == 3) S2D2_MID_BODY(3);
  else S2D2_MID_BODY(4);
#undef S2D2_MID_BODY
}

// The lines against the neighbours (us per launch, weights from memory; this kernel / the other one):
//   16 rows and fewer, where no more than 32 are possible, stay with the streaming kernel: 1.7B-shaped layer 37 / 32 (QKV, output, gate / up, down added up)
//   32 rows: 55 / 84 against two row tiles of the streaming kernel, 4B-shaped layer
//   48 rows: 66 / 64 (4B), 41 / 41 (1.7B), 97 / 97 (8B) against gemm_block.hip, 64 rows: 76 / 68, 46 / 44, 116 / 100
//   unembedding of the vocabularies that gemm_lds.hip leaves, 64 rows, less than the tiled kernel takes: 8192 features of 2048 columns 21, of 1024 14, 4096 of 2048 10
//   at most 16 rows expected, but room for more than the streaming kernel takes (a right-shifted verifier of 11 to 16 masked
//   positions; whole forwards of 12 rows, this / the streaming / the tiled kernel): 1.7B 1467 / 1439 / 3115, 4B 2423 / 2660 / 4607, 8B 3566 / 3535 / 5880
bool gemm_mid_takes(int kind, const GemmStreamArgs& a, int m_cap) {
  if (a.x_lo != LO_F16P || a.coop_wgs < 1 || a.KT % 4 || a.KT < 4 * MID_NW || a.m_hint < 1 || (a.m_hint <= 16 && m_cap <= STREAM_MOST_ROWS)) return false;
  return kind != SEPI_STORE_F32 ? a.m_hint <= MID_MOST_ROWS : a.m_hint <= 64 && (a.NT > 8 || a.gather);   // (a matrix of a few feature tiles: see the streaming kernel's launcher)
}

template <int EPI, int TPW, bool SHARED>
static void launch_mid_as(hipStream_t st, const GemmStreamArgs& a, int wgs, int passes, int KS) {
  const unsigned lds = 512 + MID_NW / 2 * MID_RB * TPW * (EPI == SEPI_SWIGLU ? 2 : 1) * 1024;
  static bool lds_set[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  if (lds > 64 * 1024 && dev >= 0 && dev < 64 && !lds_set[dev] &&
      hipFuncSetAttribute((const void*)gemm_mid_kernel<EPI, TPW, SHARED>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess)
    lds_set[dev] = true;   // on failure the launch below fails too, and the entry point reports that error
  S2D2_LAUNCH((gemm_mid_kernel<EPI, TPW, SHARED>), dim3(wgs, passes), dim3(MID_NW * 64), lds, st, a, KS);
}

template <int EPI, int TPW>
static void launch_mid(hipStream_t st, const GemmStreamArgs& a, int passes, int KS) {
  const int groups = (a.NT + TPW - 1) / TPW;
  if constexpr (EPI != SEPI_STORE_F32)
    if (KS > 1) return launch_mid_as<EPI, TPW, true>(st, a, groups * KS, passes, KS);
  launch_mid_as<EPI, TPW, false>(st, a, std::min(groups, a.coop_wgs), passes, 1);
}

// Feature tiles per workgroup (of each matrix) and workgroups that share K, by a model of the launch fitted to timings
// of all three dense models' matrices at 20, 64 and 128 rows (it is within 15 % of most of them): the larger of what
// memory and L2 deliver in all (6 and 20 TB/s, not overlapped) and to the busiest compute unit (30 and 100 GB/s), the
// merge of the wavefronts' sums, and 2.5 us for handing sums over.
static void mid_shape(int kind, const GemmStreamArgs& a, int passes, int& tpw, int& KS) {
  const int nacc = kind == SEPI_SWIGLU ? 2 : 1, rb = std::min(MID_RB, (a.m_hint + 15) / 16);
  // (what the accumulators and two tiles of operands in flight leave of 256 registers)
  const int most = kind == SEPI_STORE_F32 ? 4 : 3;
  double best = 1e30;
  tpw = KS = 1;
  for (int t = 1; t <= most; ++t)
    for (int k = 1; k <= 4; ++k) {
      const int groups = (a.NT + t - 1) / t, ta = t * nacc;
      if (k > 1 && (kind == SEPI_STORE_F32 || groups * k > a.coop_wgs || a.KT < 4 * MID_NW * k || !a.pair_buf ||
                    (long long)groups * passes * 3 * MID_RB * ta > a.pair_cap)) break;
      const double rounds = (groups * k + a.coop_wgs - 1) / a.coop_wgs, w = ta * a.KT * 1.024e-3, x = rb * a.KT * 1.024e-3;   // MB of a group
      const double us = std::max(groups * (w / 6.0 + x / 20.0), rounds / k * (w * 1e3 / 30.0 + x * 1e3 / 100.0)) + rounds * 0.12 * rb * ta + (k > 1 ? 2.5 : 0.0);
      if (us < best) { best = us; tpw = t; KS = k; }
    }
}

template <int EPI>
static void launch_mid_kind(hipStream_t st, const GemmStreamArgs& a, int m_cap) {
  const int passes = (m_cap + 16 * MID_RB - 1) / (16 * MID_RB);
  int tpw, KS;
  mid_shape(EPI, a, passes, tpw, KS);
  if constexpr (EPI == SEPI_STORE_F32) { if (tpw == 4) return launch_mid<EPI, 4>(st, a, passes, KS); }
  if (tpw == 3) return launch_mid<EPI, 3>(st, a, passes, KS);
  if (tpw == 2) return launch_mid<EPI, 2>(st, a, passes, KS);
  launch_mid<EPI, 1>(st, a, passes, KS);
}

void launch_gemm_mid(hipStream_t st, int kind, const GemmStreamArgs& a, int m_cap) {
  switch (kind) {
    case SEPI_QKV_ROPE: launch_mid_kind<SEPI_QKV_ROPE>(st, a, m_cap); break;
    case SEPI_ADD_F32: launch_mid_kind<SEPI_ADD_F32>(st, a, m_cap); break;
    case SEPI_SWIGLU: launch_mid_kind<SEPI_SWIGLU>(st, a, m_cap); break;
    case SEPI_STORE_F32: launch_mid_kind<SEPI_STORE_F32>(st, a, m_cap); break;
  }
}

}  // namespace s2d2
