// GEMM on the packed weights for windows of more than 48 rows:
//   Y[m, n] = sum_k X[m, k] W[n, k],  half operands, X in fragment order (LO_F16P).
//
// A workgroup of four wavefronts takes a block of RB x TA units of 16 x 16 and all of K (or, for narrow matrices, one of KS
// shares of K): the wavefronts split K, every operand goes straight from memory to a matrix instruction (both operands
// lie in memory in register order: 1 KB per load), no LDS and no barrier in the K loop, and the wavefronts' sums meet in LDS
// once, at the end.  The row tiles of a column sit next to each other on one XCD, so that its weights come in from memory once.
//
// What bounds it is the vector-memory path of a compute unit: requests are answered in order, about 125 to 150 GB/s while
// everything hits L2, 60 GB/s for a stream from memory whatever is in flight (4, 8 and 16 KB per wavefront, plain,
// non-temporal and coherent loads: the same), and 70 GB/s for the mixture a block reads, i.e. (RB + TA) KB per K tile of 32.
// That makes the time per K tile a property of the block's shape (below), not of the matrix, the rows or the number
// of tiles in flight, and the block's shape a choice between few bytes per unit (large blocks) and a full chip (small ones).
// (The launches of the tiled kernel are split over K and merged through memory to fill the chip; gemm_block_takes has both
// sides.)
//
#include "gemm_epilogue.h"
#include "../../include/s2d2.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace s2d2 {

static constexpr int BLK_NW = 4, BLK_THREADS = BLK_NW * 64;
static constexpr int BLK_ROW_LDS = 512 + 48 * 64;   // per-row and per-unit data in front of the sums
// K tiles in flight per wavefront: what fits next to the accumulators (two workgroups per compute unit, 256 registers;
// one with 512 from 36 units on).  More than two changed nothing (see above); the small blocks' loops are shorter with four.
constexpr int blk_u(int RB, int TA) { return RB * TA <= 16 ? 4 : 2; }
constexpr bool blk_shares(int RB, int TA) { return RB * TA != 32 && RB != 6; }   // may share K (8 x 4 has no registers for it; six row blocks are taken where they fill the chip without)
constexpr int blk_wgs(int RB, int TA) { return RB * TA > 32 ? 1 : 2; }   // workgroups per compute unit

// LDS accesses of this wavefront done, then the workgroup's barrier; global loads stay in flight.
__device__ __forceinline__ void blk_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ int blk_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(l));
  return l;
}

// Buffer loads: an operand's place is a scalar offset, a step along K inside a batch an immediate one, and the refills
// behind a share's last tile are sent out of range, where they cost an instruction and no memory access (a branch around
// them would make the compiler wait for every load in flight, a second copy of the products copies all accumulators).
constexpr uint32_t BLK_NOWHERE = 0xfffff000u;   // lane offset out of range of any matrix
struct BlkBuffers { __amdgpu_buffer_rsrc_t w, w2, x; };

template <int NACC, int TPW, int U, bool STREAM>
__device__ __forceinline__ void blk_load_w(const BlkBuffers& b, u32x4_t (&w)[TPW * NACC][U], const uint32_t (&wo)[TPW], int u, int k0, uint32_t at) {
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    w[t * NACC][u] = __builtin_amdgcn_raw_buffer_load_b128(b.w, at + u * 1024, wo[t] + (uint32_t)k0 * 1024u, STREAM ? 2 : 0);
    if (NACC == 2) w[t * NACC + 1][u] = __builtin_amdgcn_raw_buffer_load_b128(b.w2, at + u * 1024, wo[t] + (uint32_t)k0 * 1024u, STREAM ? 2 : 0);
  }
}

// Row tiles pass, pass + rows_t, .. of 16 RB rows (RBX: most of the launch); w holds the first U tiles of the share.
template <int EPI, int RB, int RBX, int TA, int U, bool SHARED, bool STREAM>
__device__ __forceinline__ void gemm_block_body(const GemmStreamArgs& a, const BlkBuffers& b, u32x4_t (&w)[TA][U], const uint32_t (&wo)[TA / (EPI == SEPI_SWIGLU ? 2 : 1)],
                                                const int n, const int kb, const int grp, const int ks, int pass, const int rows_t, const int M,
                                                const int groups, const int KS, uint8_t* smem) {
  constexpr int NACC = EPI == SEPI_SWIGLU ? 2 : 1, TPW = TA / NACC, NU = RB * TPW, HW = BLK_NW / 2;
  constexpr bool AGPR = blk_wgs(RBX, TA) == 1;   // accumulators in the upper half of 512 registers (left to itself the compiler copies them to and fro: 288 of 473 instructions in the K loop)
  float* s_rs = (float*)smem;                       // [128] 1/rms of the rows
  int2* s_seq = (int2*)(smem + 512);                // [128] sequence of a row and the sequence's first row
  float* s_sq = (float*)(smem + 512);               // [units][16] sums of squares (residual add)
  f32x4_t* s_red = (f32x4_t*)(smem + BLK_ROW_LDS);  // [wavefront of a half][unit][accumulator][lane]
  // (opaque: what depends on the thread index alone is otherwise computed ahead of the switch for all row counts and kept)
  const int lane = blk_lane(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane16 = lane * 16;
  const int KT = a.KT;
  u32x4_t x[RB][U];
  for (;;) {
    const int m0 = pass * RB * 16, Mloc = min(RB * 16, M - m0);
    uint32_t xo[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)   // blocks past the rows read the last one again; never stored
      xo[rb] = ((uint32_t)min((m0 >> 4) + rb, (M - 1) >> 4) * (uint32_t)KT + (uint32_t)kb) * 1024u;
    auto load_x = [&](int u, int k0, uint32_t at) __attribute__((always_inline)) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) x[rb][u] = __builtin_amdgcn_raw_buffer_load_b128(b.x, at + u * 1024, xo[rb] + (uint32_t)k0 * 1024u, 0);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) load_x(u, 0, lane16);
    __builtin_amdgcn_sched_barrier(0);

    f32x4_t acc[RB][TA];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int t = 0; t < TA; ++t) acc[rb][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mac = [&](int u) __attribute__((always_inline)) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < TA; ++t) {
          if (AGPR) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc[rb][t]) : "v"(w[t][u]), "v"(x[rb][u]));
          else acc[rb][t] = mfma_16x16x32<OPM_F16>(w[t][u], x[rb][u], acc[rb][t]);
        }
    };
    if (AGPR) asm volatile("s_nop 7");   // (cleared accumulators, ahead of the first product)
    // sliding window over the K tiles: a slot is refilled right after its last use
    int k0 = 0;
    do {
      k0 += U;
      const uint32_t at = k0 < n ? lane16 : BLK_NOWHERE;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        mac(u);
        blk_load_w<NACC, TPW, U, STREAM>(b, w, wo, u, k0, at);
        load_x(u, k0, at);
        __builtin_amdgcn_sched_barrier(0);   // (the scheduler otherwise gathers the batch's loads behind its products)
      }
    } while (k0 < n);
    if (AGPR) {   // the results are there (the compiler does not know what these instructions are)
      asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < TA; ++t) asm volatile("" : "+a"(acc[rb][t]));
    }

    // ---- the wavefronts' sums, through LDS: the upper two add theirs to the lower two's, then every wavefront sums its
    // units (wave, wave + 4, ...) over the two.  What the epilogue reads (residual, gains, rotations) is requested ahead of
    // the second barrier (ahead of the first the accumulators leave no registers). ----
    const int lm = blk_lane();   // (not kept in a register across the K loop)
    const int gm = lm >> 4, fm = lm & 15;
    if (wave >= HW) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < TA; ++t) s_red[(((wave - HW) * RB + rb) * TA + t) * 64 + lm] = acc[rb][t];
    }
    blk_barrier();
    if (wave < HW) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int t = 0; t < TA; ++t) {
          f32x4_t* p = &s_red[((wave * RB + rb) * TA + t) * 64 + lm];
          *p = acc[rb][t] + *p;
        }
    } else if (EPI != SEPI_ADD_F32) {
      // the others: 1/rms of the rows from the producer's partial sums of squares (in front of the K loop it kept the
      // first multiplication waiting: gate / up, 8B shape, 512 rows, 141 us for 155), and the rows' sequences
      constexpr int TPR = RB == 2 ? 4 : RB <= 4 ? 2 : 1, SSV = 8;   // threads per row, float4 per thread and round
      const int ht = (wave - HW) * 64 + lm, ss_row = ht / TPR, ss_sub = ht % TPR;
      const int rr = min(m0 + ss_row, M - 1);   // rows past the count read a valid row; their 1/rms is never used
      const int seq = EPI == SEPI_QKV_ROPE ? a.row_seq[rr] : 0;
      const float* pp = a.ss_part + (size_t)rr * a.ss_stride;
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
      if (ss_row < RB * 16 && ss_sub == 0) {
        s_rs[ss_row] = 1.0f / sqrtf(v / (float)a.K + a.eps);
        if (EPI == SEPI_QKV_ROPE) s_seq[ss_row] = make_int2(seq, a.seq_row0[seq]);
      }
    }
    auto unit = [&](int q) __attribute__((always_inline)) { return wave + BLK_NW * q; };   // of this wavefront
    constexpr int UPW = (NU + BLK_NW - 1) / BLK_NW;
    struct Ahead { float4 h; EpiAhead e; };
    auto request = [&](int u, Ahead& n_) __attribute__((always_inline)) {
      if (EPI == SEPI_SWIGLU) return;
      u = min(u, NU - 1);   // (places that do not exist read a valid one)
      const int r = min(m0 + (u / TPW) * 16 + fm, M - 1), nt = min(grp * TPW + u % TPW, a.NT - 1);
      gemm_epi_request<EPI>(a, r, nt, gm, n_.e);
      if (EPI == SEPI_ADD_F32) n_.h = *(const float4*)((const float*)a.out + (size_t)r * a.ldo + nt * 16 + 4 * gm);
    };
    constexpr int DEP = EPI == SEPI_SWIGLU ? 1 : 3;   // units requested ahead
    Ahead next[DEP];
    if (!SHARED) {
#pragma unroll
      for (int i = 0; i < DEP; ++i) request(unit(i), next[i]);
    }
    blk_barrier();
    auto unit_sum = [&](int u, f32x4_t (&sum)[NACC]) __attribute__((always_inline)) {
#pragma unroll
      for (int c = 0; c < NACC; ++c) {
        const f32x4_t* p = &s_red[(u * NACC + c) * 64 + lm];
        sum[c] = p[0] + p[NU * NACC * 64];
      }
    };
    auto unit_ok = [&](int u) __attribute__((always_inline)) {   // uniform over the wavefront
      return u < NU && (u / TPW) * 16 < Mloc && grp * TPW + u % TPW < a.NT;
    };
    auto finish = [&](int u, const f32x4_t (&sum)[NACC], Ahead& at) __attribute__((always_inline)) {
      const int r = (u / TPW) * 16 + fm;
      float sq = 0.f;
      if (EPI == SEPI_QKV_ROPE) { const int2 sr = s_seq[r]; at.e.seq = sr.x; at.e.row0 = sr.y; }
      gemm_epi_unit<EPI, true>(a, r < Mloc, m0 + min(r, Mloc - 1), EPI == SEPI_ADD_F32 ? 1.0f : s_rs[r], grp * TPW + u % TPW, gm, sum[0], sum[NACC - 1], &at.h, &sq, &at.e);
      if (EPI == SEPI_ADD_F32 && gm == 0) s_sq[u * 16 + fm] = sq;
    };
    // (Loops over units are not unrolled: that is 10-20 KB of instructions that every workgroup would fetch once.)
    if (!SHARED) {
#pragma unroll 1
      for (int q0 = 0; q0 < UPW; q0 += DEP) {
#pragma unroll
        for (int i = 0; i < DEP; ++i) {
          const int u = unit(q0 + i);
          if (unit_ok(u)) {
            f32x4_t sum[NACC];
            unit_sum(u, sum);
            finish(u, sum, next[i]);
          }
          request(unit(q0 + i + DEP), next[i]);
        }
      }
    } else {
      // K shared by KS workgroups: the shares 1 .. KS - 1 (first in dispatch order; they never wait) hand their sums over as
      // 64-bit (value, tag) words; share 0 requests the words of a batch of units from all of them until all are there,
      // adds them in share order, clears them for the next launch and finishes the units.  The wait is bounded; one
      // that runs out sets *pair_status and goes on with what is there.
      static_assert(!SHARED || NACC == 1, "one accumulator per unit");
      constexpr int KSM = 4, BU = NU > 16 ? 2 : UPW < 4 ? UPW : 4;   // units per batch: 24 registers of words each
      unsigned long long* slot0 = a.pair_buf + (size_t)(pass * groups + grp) * (KS - 1) * (RBX * TPW) * 256 + lm;   // [row tile][group][share - 1][unit]
      if (ks > 0) {
#pragma unroll 1
        for (int q = 0; q < UPW; ++q) {
          const int u = unit(q);
          if (!unit_ok(u)) continue;
          f32x4_t sum[NACC];
          unit_sum(u, sum);
          unsigned long long* slot = slot0 + ((size_t)(ks - 1) * NU + u) * 256;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            __hip_atomic_store(slot + i * 64, (unsigned long long)__float_as_uint(sum[0][i]) | (1ull << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      } else {
#pragma unroll 1
        for (int q0 = 0; q0 < UPW; q0 += BU) {
          Ahead at[BU];
#pragma unroll
          for (int j = 0; j < BU; ++j) request(unit(q0 + j), at[j]);
          int first = -1;   // a unit of the batch that is there
#pragma unroll
          for (int j = BU - 1; j >= 0; --j)
            if (q0 + j < UPW && unit_ok(unit(q0 + j))) first = unit(q0 + j);
          if (first < 0) continue;   // (no rows)
          unsigned long long v[BU][KSM - 1][4];
          int spins = 0;
          for (; spins < (1 << 20); ++spins) {
            unsigned long long all = ~0ull;
#pragma unroll
            for (int j = 0; j < BU; ++j) {
              int u = unit(q0 + j);
              if (q0 + j >= UPW || !unit_ok(u)) u = first;   // not there: another one again
#pragma unroll
              for (int k = 0; k < KSM - 1; ++k) {
                const unsigned long long* slot = slot0 + ((size_t)min(k, KS - 2) * NU + u) * 256;   // (fewer shares: the last one again)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[j][k][i] = __hip_atomic_load(slot + i * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
            }
#pragma unroll
            for (int j = 0; j < BU; ++j)
#pragma unroll
              for (int k = 0; k < KSM - 1; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) all &= v[j][k][i];
            if (all >> 32) break;
          }
          if (spins == (1 << 20) && a.pair_status) *a.pair_status = 1;
#pragma unroll
          for (int j = 0; j < BU; ++j) {
            const int u = unit(q0 + j);
            if (q0 + j >= UPW || !unit_ok(u)) continue;
            f32x4_t sum[NACC];
            unit_sum(u, sum);
#pragma unroll
            for (int k = 0; k < KSM - 1; ++k) {
              if (k >= KS - 1) break;   // uniform
              unsigned long long* slot = slot0 + ((size_t)k * NU + u) * 256;
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                __hip_atomic_store(slot + i * 64, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sum[0][i] += __uint_as_float((uint32_t)v[j][k][i]);
              }
            }
            finish(u, sum, at[j]);
          }
        }
      }
    }
    if (EPI == SEPI_ADD_F32 && ks == 0 && a.ss_out) {
      // the rows' sums of squares over the group's features, one number each (a quarter of the consumers' reads or less);
      // the last group also clears the entries that round their number up
      blk_barrier();
      const int r = wave * 64 + lm;
      if (r < Mloc) {
        float v = 0.f;
#pragma unroll
        for (int t = 0; t < TPW; ++t) v += grp * TPW + t < a.NT ? s_sq[((r >> 4) * TPW + t) * 16 + (r & 15)] : 0.f;
        float* p = a.ss_out + (size_t)(m0 + r) * a.ss_stride;
        p[grp] = v;
        if (grp == groups - 1)
          for (int i = groups; i < min((groups + 3) & ~3, a.ss_stride); ++i) p[i] = 0.f;
      }
    }
    pass += rows_t;
    if (pass * RB * 16 >= M) break;
    // rows beyond the expected ones: the same columns again
    blk_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u) blk_load_w<NACC, TPW, U, STREAM>(b, w, wo, u, 0, lane16);
  }
}


// P row tiles expected.  The row count is on the device: tiles shrink with it (compiled for a few of them), so that a launch
// of fewer rows still fills the chip; workgroups without rows are the last ones.
template <int EPI, int RB, int TA, bool SHARED, bool STREAM>
__global__ __launch_bounds__(BLK_THREADS, blk_wgs(RB, TA)) void gemm_block_kernel(const GemmStreamArgs a, const int P, const int groups, const int KS_, const int rows_max) {
  constexpr int NACC = EPI == SEPI_SWIGLU ? 2 : 1, TPW = TA / NACC, U = blk_u(RB, TA);
  static_assert(TA % NACC == 0, "gate and up tiles come in pairs");
  extern __shared__ __align__(16) uint8_t smem[];
  const int KT = a.KT, KS = SHARED ? KS_ : 1;
  const uint32_t wbytes = (uint32_t)a.NT * (uint32_t)KT * 1024u, xbytes = (uint32_t)((rows_max + 15) >> 4) * (uint32_t)KT * 1024u;
  const BlkBuffers b = {__builtin_amdgcn_make_buffer_rsrc((void*)a.Wp, 0, wbytes, 0x00020000),
                        __builtin_amdgcn_make_buffer_rsrc((void*)(NACC == 2 ? a.Wp2 : a.Wp), 0, wbytes, 0x00020000),
                        __builtin_amdgcn_make_buffer_rsrc((void*)a.X, 0, xbytes, 0x00020000)};
  // XCD i % 8 owns the columns (groups of TPW feature tiles) c % 8 == i % 8: per share of K (the ones that hand their
  // sums over first), all row tiles of a column next to each other.
  const int cols = (groups + 7) >> 3, xcd = blockIdx.x & 7, s_ = (int)blockIdx.x >> 3;
  int rows_t = P, ks = 0, grp = 0, pass = 0, n = 0, kb = 0;
  uint32_t wo[TPW];   // the group's weight tiles, first K tile of this wavefront
  u32x4_t w[TA][U];
  auto place = [&]() __attribute__((always_inline)) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (scalar: K bounds must give scalar branches)
    const int per = cols * rows_t, sh = SHARED ? s_ / per : 0, q = s_ - sh * per;
    ks = KS - 1 - sh;
    grp = (q / rows_t) * 8 + xcd;
    pass = q % rows_t;
    const int share = ks * BLK_NW + wave, nb = KT / U, parts = BLK_NW * KS;
    kb = share * nb / parts * U;
    n = (share + 1) * nb / parts * U - kb;   // whole batches of U tiles, at least one
#pragma unroll
    for (int t = 0; t < TPW; ++t) wo[t] = ((uint32_t)min(grp * TPW + t, a.NT - 1) * (uint32_t)KT + (uint32_t)kb) * 1024u;
    const uint32_t lane16 = blk_lane() * 16;
#pragma unroll
    for (int u = 0; u < U; ++u) blk_load_w<NACC, TPW, U, STREAM>(b, w, wo, u, 0, lane16);
  };
  place();   // the weights of the first tiles, placed as if the rows were the expected ones: their addresses need no row count
  const int M = *a.m_count, blocks = (M + 15) >> 4, rb = (blocks + P - 1) / P;   // 16-row blocks of a tile
  if (blocks == 0) return;
  auto run = [&](auto rb_tag) __attribute__((always_inline)) {
    constexpr int R = decltype(rb_tag)::value;
    const int tiles = (blocks + R - 1) / R;
    if (tiles < P) {   // fewer: workgroups without rows are the last ones
      rows_t = tiles;
      if (s_ >= cols * rows_t * KS) return;
      place();
    }
    if (grp >= groups) return;
    gemm_block_body<EPI, R, RB, TA, U, SHARED, STREAM>(a, b, w, wo, n, kb, grp, ks, pass, rows_t, M, groups, KS, smem);
  };
  if ((RB == 8 && rb > 6) || (RB == 6 && rb > 4) || (RB == 4 && rb > 3) || (RB == 2 && rb > 1)) run(std::integral_constant<int, RB>{});
  else if (RB == 8 && rb > 4) run(std::integral_constant<int, 6>{});
  else if (RB >= 6 && rb > 3) run(std::integral_constant<int, 4>{});
  else if (RB >= 4 && rb > 2) run(std::integral_constant<int, 3>{});
  else if (RB >= 4 && rb > 1) run(std::integral_constant<int, 2>{});
  else run(std::integral_constant<int, 1>{});
}

// ---- choice of the block ----
// Time per K tile (of 32) and, behind it, time of a workgroup's ends, us: K 4096 and 12288, 64 to 512 rows, one workgroup per
// compute unit.
struct BlkShape { int rb, ta; double per_kt, ends; };
static constexpr BlkShape BLK_SHAPES[] = {{2, 2, .066, 3.0}, {4, 2, .092, 3.2}, {4, 3, .104, 3.6}, {4, 4, .115, 3.9}, {4, 6, .141, 4.9}, {6, 4, .146, 4.9},
                                          {8, 4, .168, 5.3}, {6, 6, .185, 8.0}, {8, 6, .205, 9.0}, {6, 8, .205, 9.0}};
struct BlkPick { int rb, ta, KS; double us; };
// Six row blocks: 768 rows of the 1.7B shape are 256 blocks of 6 x 4 in the output and down projection (192 of 8 x 4: 56 -> 47 us for the
// two, with the requests of the epilogue) and of 6 x 8 in QKV (768 of 4 x 4, two or three on a compute unit: 32.8 -> 28.8).  From 56 K tiles on: forwards of four layers of
// 704 to 1536 rows without / with them 1792 columns 983 / 951 to 678 / 663 us, 1920 686 / 673; at 1536 columns the difference is less than the estimates below are off by (0.993 to
// 1.011 of the time), and the other shapes stay.
constexpr bool blk_compiled(int kind, int RB, int TA) {
  return kind == SEPI_SWIGLU ? TA != 3 && TA != 8 : RB == 6 ? TA == 8 || (TA == 4 && kind == SEPI_ADD_F32) : true;
}

// A launch takes the longer of what its busiest compute unit and what the chip needs: rounds of workgroups times the times
// above (where two workgroups share a compute unit and there are several rounds, most of a workgroup's ends is hidden), and the weights from memory at 6.3 TB/s, then the rest of the operands from L2 at 25, behind 3 us; activations that do not stay in an XCD's L2 are
// read once per column of blocks at 9 (1.7B down projection, 4992 rows: 279 us for the 178 of the tiled kernel).  Of 72 cases (three
// dense models' matrices, 64 to 512 rows) the block it picks is 1.3 % slower than the fastest on average.
// Sharing K costs 2.5 us for the hand-over and 0.3 for each unit (2 KB of words per share, through memory).
static BlkPick blk_pick(int kind, const GemmStreamArgs& a, int m_cap) {
  BlkPick best{0, 0, 1, 1e30};
  const int nacc = kind == SEPI_SWIGLU ? 2 : 1;
  const double kt_mb = 1.024e-3;   // MB of a unit's operand per K tile
  for (const BlkShape& s : BLK_SHAPES) {
    if (s.ta % nacc || !blk_compiled(kind, s.rb, s.ta) || (kind != SEPI_SWIGLU && s.rb == 6 && a.KT < 56)) continue;
    const int tpw = s.ta / nacc, groups = (a.NT + tpw - 1) / tpw, tiles = (a.m_hint + 16 * s.rb - 1) / (16 * s.rb), caps = (m_cap + 16 * s.rb - 1) / (16 * s.rb);
    const int u = blk_u(s.rb, s.ta);
    for (int ks = 1; ks <= 4; ++ks) {
      if (ks > 1 && (kind != SEPI_ADD_F32 || !blk_shares(s.rb, s.ta) || !a.pair_buf || (groups + 7) / 8 * 8 * tiles * ks > a.coop_wgs || (long long)groups * caps * (ks - 1) * s.rb * tpw > a.pair_cap)) break;
      if (a.KT % u || a.KT / u < BLK_NW * ks) break;
      const double rounds = (groups + 7) / 8 * tiles * ks / (a.coop_wgs / 8.0);   // of the compute units of an XCD
      const double work = a.KT * s.per_kt / ks;
      const double cu = (blk_wgs(s.rb, s.ta) == 1 || rounds <= 2 ? std::ceil(rounds) * (work + s.ends) : 0.5 * (rounds + std::ceil(rounds)) * (work + 0.3 * s.ends) + s.ends) +
                        (ks > 1 ? 2.5 + 0.3 * (s.rb * tpw) : 0.0);
      const double w = (double)a.NT * nacc * a.KT * kt_mb, x = (double)groups * tiles * (s.rb + s.ta) * a.KT * kt_mb - w;
      const double rows_mb = a.m_hint * a.KT * 64e-6;   // the activations
      const double us = std::max(std::max(cu, w / 6.3 + x / 25.0 + 3.0), rows_mb > 3.0 ? groups * rows_mb / 9.0 : 0.0);
      if (us < best.us) best = {s.rb, s.ta, ks, us};
    }
  }
  return best;
}

template <int EPI, int RB, int TA, bool SHARED, bool STREAM>
static int launch_blk(hipStream_t st, const GemmStreamArgs& a, int KS, int m_cap) {
  constexpr int TPW = TA / (EPI == SEPI_SWIGLU ? 2 : 1);
  constexpr unsigned lds = BLK_ROW_LDS + BLK_NW / 2 * RB * TA * 1024;
  static bool lds_set[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  if (lds > 64 * 1024 && dev >= 0 && dev < 64 && !lds_set[dev] &&
      hipFuncSetAttribute((const void*)gemm_block_kernel<EPI, RB, TA, SHARED, STREAM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess)
    lds_set[dev] = true;   // on failure the launch below fails too, and the entry point reports that error
  const int passes = (a.m_hint + 16 * RB - 1) / (16 * RB), groups = (a.NT + TPW - 1) / TPW;
  S2D2_LAUNCH((gemm_block_kernel<EPI, RB, TA, SHARED, STREAM>), dim3((groups + 7) / 8 * 8 * passes * KS), dim3(BLK_THREADS), lds, st, a, passes, groups, KS, m_cap);
  return std::min((groups + 3) & ~3, a.ss_stride);
}

// Streaming loads leave what the next kernels need in L2 (their code, the plan, the rows that this one writes): with plain loads
// the 1.7B attention behind the QKV projection takes 16.4 us for 15.0, an embedding launch 8.3 for 7.6.  Where more row tiles read the
// same weights again they cost more than that (256 rows 4B: down projection 36.5 -> 38.5, 128 rows 1.7B 15.5 -> 16.0).
constexpr bool blk_streams(int kind, int RB, int TA) { return RB <= 4 || (kind == SEPI_SWIGLU && TA == 6); }   // compiled; up to 64 rows the pick has four row blocks or fewer in all other shapes
static bool blk_stream(int kind, const BlkPick& p, int rows) {
  return blk_streams(kind, p.rb, p.ta) && rows <= (kind == SEPI_SWIGLU && p.ta == 6 && p.rb > 4 ? 16 * p.rb : 64);
}

template <int EPI, int RB, int TA>
static int launch_blk_shape(hipStream_t st, const GemmStreamArgs& a, const GemmChoice& c, int m_cap) {
  if constexpr (EPI == SEPI_ADD_F32 && blk_shares(RB, TA)) {
    if constexpr (blk_streams(EPI, RB, TA))
      if (c.KS > 1 && c.stream) return launch_blk<EPI, RB, TA, true, true>(st, a, c.KS, m_cap);
    if (c.KS > 1) return launch_blk<EPI, RB, TA, true, false>(st, a, c.KS, m_cap);
  }
  if constexpr (blk_streams(EPI, RB, TA))
    if (c.stream) return launch_blk<EPI, RB, TA, false, true>(st, a, 1, m_cap);
  return launch_blk<EPI, RB, TA, false, false>(st, a, 1, m_cap);
}

template <int EPI>
static int launch_blk_kind(hipStream_t st, const GemmStreamArgs& a, const GemmChoice& c, int m_cap) {
#define S2D2_BLK(RB, TA) if (c.rb == RB && c.ta == TA) return launch_blk_shape<EPI, RB, TA>(st, a, c, m_cap)
  S2D2_BLK(2, 2); S2D2_BLK(4, 2); S2D2_BLK(4, 4); S2D2_BLK(4, 6); S2D2_BLK(8, 4); S2D2_BLK(8, 6);
  if constexpr (EPI == SEPI_SWIGLU) { S2D2_BLK(6, 4); S2D2_BLK(6, 6); }
  else { S2D2_BLK(4, 3); S2D2_BLK(6, 8); if constexpr (EPI == SEPI_ADD_F32) { S2D2_BLK(6, 4); } }
#undef S2D2_BLK
  return 0;   // (the pick is one of these)
}

// Wider than the mid-size kernel's windows, and faster than the tiled kernel by its launcher's estimate and this one's.  The latter is
// 1.1 times too short on average for the products inside a forward (where the epilogue and operands that the kernel before
// has just written count as well).  Inside forwards, us per launch, this kernel / the tiled one: QKV 8B 256 rows 32 / 44, 512
// 48 / 54, 4B 22 / 35, 35 / 43, 1.7B 512 rows 22 / 35, MoE 1024 rows 32 / 40; output 8B 23 / 35, 34 / 39, 4B 18 / 29, 27 / 45, 1.7B
// 14 / 28, MoE 21 / 35; down 8B 56 / 69, 4B 37 / 43, 51 / 68, 1.7B 29 / 35; gate / up 4B 512 rows 71 / 85, 128 rows 34 / 45, 1.7B 128
// rows 18 / 26, 8B 96 rows 46 / 58, and left to others 8B 256 rows 82 / 73, 512 141 / 109, 4B 256 53 / 46, 1.7B 512 43 / 36 (gate / up of so many rows goes through LDS
// now, see gemm_lds.hip).
bool gemm_block_takes(int kind, const GemmStreamArgs& a, int m_cap, GemmChoice& c) {
  if (a.x_lo != LO_F16P || a.coop_wgs < 1 || a.KT % 4 || a.KT < 4 * BLK_NW || a.m_hint <= MID_MOST_ROWS || a.grouped != GROUP_NONE || kind == SEPI_STORE_F32) return false;
  if ((long long)a.NT * a.KT * 1024 >= 1LL << 32 || (long long)(m_cap + 15) / 16 * a.KT * 1024 >= 1LL << 32) return false;   // (32-bit offsets)
  const BlkPick p = blk_pick(kind, a, m_cap);
  if (p.rb == 0 || 1.1 * p.us >= gemm_tile_us(kind, a, (m_cap + 127) / 128) || (kind == SEPI_SWIGLU && 1.1 * p.us >= gemm_lds_gateup_us(a))) return false;
  c = {GEMM_BLOCK, p.rb, p.ta, p.KS, blk_stream(kind, p, a.m_hint)};
  return true;
}

int launch_gemm_block(hipStream_t st, int kind, const GemmStreamArgs& a, int m_cap, const GemmChoice& c) {
  switch (kind) {
    case SEPI_QKV_ROPE: return launch_blk_kind<SEPI_QKV_ROPE>(st, a, c, m_cap);
    case SEPI_ADD_F32: return launch_blk_kind<SEPI_ADD_F32>(st, a, c, m_cap);
    case SEPI_SWIGLU: return launch_blk_kind<SEPI_SWIGLU>(st, a, c, m_cap);
  }
  return 0;
}

}  // namespace s2d2
