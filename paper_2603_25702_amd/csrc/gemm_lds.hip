// GEMMs on the packed weights with both operands through LDS, half operands:
//   Y[m, n] = sum_k X[m, k] W[n, k]   for the unembedding of more than 16 rows, and for the rows of one expert of the MoE FFN (X in rows).
//
// A workgroup of eight wavefronts takes up to 256 rows x 256 features (128 of gate and up each) and all of K: up to 256 rows, and for most experts,
// the weights are requested once.  Both operands go from memory into LDS without a register on the way (a wavefront's
// request is 1 KB; rows are gathered by the lanes' addresses), and every wavefront multiplies half of the row blocks with a quarter of the
// features.  The reads of the next 32 columns and the requests to come are issued one by one between the matrix instructions (left to the
// compiler all reads of a step come first: 92 us for 73 of a dense product of 256 rows, K 4096).
//
// What bounds it: a compute unit's requests are answered in order, about 400 lines a microsecond while the weights come from memory, whatever is in
// flight; and all weights together at 6 to 7 TB/s.  (Bringing lines into L2 ahead of time takes the same places in that order: slower.)
// The tiled kernel asks for 1.5 times the lines, and for the weights of an expert with 130 rows twice.  64 experts of 2048 x 1024, launches alone, us, tiled
// kernel / this one: gate / up, 18 rows an expert on average 103 / 81 (6.6 TB/s), 64 rows 110 / 89, 128 rows 131 / 110, the most chosen with
// 700 144 / 135; down 72 / 47, 89 / 56, 108 / 68, 108 / 80.  Inside the draft of 32 sequences of 32, 128 rows an expert on average, this kernel takes 121 to 126 and 76 to 78.
//
// One workgroup per compute unit takes tile after tile: XCD x those of the experts that moe_group_kernel gave it (of a slice of their features, where there are few experts), the largest
// first and in alternating order, so that a workgroup's tiles add up to about the same rows.  The first requests of a workgroup's next tile are made ahead of
// the stores of the present one (launches of a workgroup per tile take 6 to 7 us longer at 128 rows).
#include "gemm_epilogue.h"
#include "../../include/s2d2.h"

#include <algorithm>
#include <type_traits>

namespace s2d2 {

static constexpr int LDS_NW = 8, LDS_THREADS = LDS_NW * 64;
static constexpr int LDS_WR = 2, LDS_WC = LDS_NW / LDS_WR, LDS_TW = 4, LDS_TA = LDS_WC * LDS_TW;   // wavefronts along rows and features; feature tiles of a wavefront and of the workgroup
static constexpr uint32_t LDS_NOWHERE = 0xfffff000u;   // lane offset out of range of any operand: an instruction, no memory access
// LDS holds a ring of the rows' 64 columns (XS places) and one of the weights' 32 (WS): by row blocks per wavefront, what fits.  Requests are answered in
// order, so either operand's lead has to cover all lines that are asked for ahead of it: rows two steps ahead behind weights that are five
// ahead take 1.17 us a step where their lines take 0.64 (256 rows).
constexpr int lds_xs(int RBL) { return RBL <= 4 ? 4 : 3; }
constexpr int lds_ws(int RBL) { return RBL <= 2 ? 6 : RBL <= 4 ? 5 : RBL <= 6 ? 4 : 3; }
static constexpr unsigned LDS_BYTES = 144 * 1024;
// Order of a wavefront's requests, by K step s of 32 columns: WL of the weights of step s + WS, and in odd steps XL of the rows of the steps
// s + 2 XS - 1 and + 2 XS.  How many of them come behind the ones that step k + 1 needs, when step k looks (by whether k is odd).
constexpr int lds_behind(int odd, int WS, int XS, int WL, int XL) {
  const int k = 64 + odd, w = k + 1 - WS, x = odd ? k + 1 - 2 * XS + 1 : -1;   // the steps that requested them
  int last = 0, at = 0;
  for (int s = 0; s < k; ++s) {
    at += WL;
    if (s == w) last = at;
    if (s & 1) {
      at += XL;
      if (s == x) last = at > last ? at : last;
    }
  }
  return at - last;
}

template <int I, int N, typename F>
__device__ __forceinline__ void lds_each(const F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    lds_each<I + 1, N>(f);
  }
}
// Sum of squares of a row from its producer's partial sums, by the two lanes sub = 0 and 1.
__device__ __forceinline__ float lds_row_squares(const GemmStreamArgs& a, int row, int sub) {
  const float* pp = a.ss_part + (size_t)row * a.ss_stride;
  float v = 0.f;
  if ((a.ss_count & 3) == 0 && (a.ss_stride & 3) == 0) {
    const int n4 = a.ss_count >> 2;
    for (int i0 = sub; i0 < n4; i0 += 16) {
      float4 t[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = ((const float4*)pp)[min(i0 + 2 * j, n4 - 1)];   // clamped duplicates are skipped when summing
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i0 + 2 * j < n4) v += (t[j].x + t[j].y) + (t[j].z + t[j].w);
    }
  } else {
    for (int i = sub; i < a.ss_count; i += 2) v += pp[i];
  }
  return v + __shfl_xor(v, 1, 64);
}
// A value that is the same in all lanes, in a scalar register for certain (a request's operands have to be).
__device__ __forceinline__ uint32_t lds_uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
// 64 lanes x 16 bytes from memory to LDS at `at` + 16 lane
template <bool STREAM>
__device__ __forceinline__ void lds_request(const __amdgpu_buffer_rsrc_t& rs, uint32_t voff, uint32_t soff, uint32_t at) {
  if (STREAM) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(at), "v"(voff), "s"(rs), "s"(soff) : "memory");
  else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(at), "v"(voff), "s"(rs), "s"(soff) : "memory");   // (the compiler keeps nothing in m0 here)
}
// at most N of this wavefront's requests outstanding, its LDS reads done; then the workgroup's barrier
template <int N>
__device__ __forceinline__ void lds_wait_barrier() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory"); }

struct LdsItem { int m0, rows, expert, nt0, tiles; };   // nt0: first feature tile (of either matrix), tiles: how many
// A tile's operands: buffers, and the places of this wavefront's units (1 KB each) of a stage
struct LdsPlaces {
  uint64_t w;       // weights of the tile's features (gate and up: a wavefront requests units of one of the two)
  uint32_t wbytes;
  uint32_t wo[2], wv[2];   // weights: scalar offset of the unit; LDS_NOWHERE if it does not exist
  uint32_t xv[4];   // rows: a lane's offset
};

struct LdsBuffers {
  __amdgpu_buffer_rsrc_t w, x;
  uint32_t wo[2], wv[2];
  __device__ __forceinline__ LdsBuffers(const GemmStreamArgs& a, const LdsPlaces& p, uint32_t xbytes) {
    w = __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)lds_uniform((uint32_t)(p.w >> 32)) << 32 | lds_uniform((uint32_t)p.w)), 0, lds_uniform(p.wbytes), 0x00020000);
    x = __builtin_amdgcn_make_buffer_rsrc((void*)a.X, 0, xbytes, 0x00020000);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      wo[i] = lds_uniform(p.wo[i]);
      wv[i] = lds_uniform(p.wv[i]);
    }
  }
};

// ROWS: X in rows, else in fragment order.  STREAM: weights past the caches.
template <int EPI, bool ROWS, bool STREAM>
struct LdsTile {
  static constexpr int NACC = EPI == SEPI_SWIGLU ? 2 : 1, TPW = LDS_TA / NACC, TWP = LDS_TW / NACC;
  static constexpr int WL = LDS_TA / LDS_NW;                             // units of a wavefront: weights (32 columns)
  static constexpr int xl(int RBL) { return 2 * LDS_WR * RBL / LDS_NW; }   // rows (8 of them, 64 columns)
  static constexpr uint32_t xplace(int RBL) { return 2 * LDS_WR * RBL * 1024u; }
  static constexpr uint32_t WPLACE = LDS_TA * 1024u;
  static constexpr uint32_t wring(int RBL) { return lds_xs(RBL) * xplace(RBL); }

  static __device__ __forceinline__ void request_w(const LdsBuffers& b, uint32_t lds0, int wave, uint32_t lane16, int i, int k, uint32_t place, bool there) {
    lds_request<STREAM>(b.w, there ? lane16 | b.wv[i] : LDS_NOWHERE, b.wo[i] + (uint32_t)k * 1024u, lds0 + place + (wave + LDS_NW * i) * 1024u);
  }
  // X in rows: eight rows' 128 bytes each, whole lines (16 rows x 64 bytes are twice as many line requests: gate / up at 64 rows an expert 95 us for 88).
  // A row's 16-byte pieces are stored in the order piece ^ (row % 8), which lets the operand reads (16 rows, one piece each) hit all banks.  In fragment order a unit is 16 rows x 32 columns as
  // the matrix instruction takes them.
  static __device__ __forceinline__ void request_x(const LdsBuffers& b, const uint32_t (&xv)[4], uint32_t lds0, int wave, int i, int k2, uint32_t place, bool there) {
    lds_request<false>(b.x, there ? xv[i] : LDS_NOWHERE, (uint32_t)k2 * (ROWS ? 128u : 2048u), lds0 + place + (wave + LDS_NW * i) * 1024u);
  }
  template <int RBL>
  static __device__ __forceinline__ void request_first(const GemmStreamArgs& a, LdsPlaces& p, const LdsBuffers& b, const LdsItem& it, const int* s_src, uint32_t lds0, int wave, int lane, int n) {
    constexpr int XL = xl(RBL), XS = lds_xs(RBL), WS = lds_ws(RBL);
    static_assert(XL >= 1 && XL <= 4 && XL * LDS_NW == 2 * LDS_WR * RBL && WL == 2 && wring(RBL) + WS * WPLACE <= LDS_BYTES, "whole units per wavefront");
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int t = wave + LDS_NW * i;
      if (ROWS) p.xv[i] = (uint32_t)s_src[(t >> 1) * 16 + (t & 1) * 8 + (lane >> 3)] * (uint32_t)a.ldx * 2u + (uint32_t)((lane & 7) ^ (lane >> 3)) * 16u;
      else p.xv[i] = 2u * (uint32_t)frag_offset(s_src[(t >> 1) * 16 + (lane & 15)], 8 * (lane >> 4), a.K) + (t & 1) * 1024u;
      if ((t >> 1) * 16 >= it.rows) p.xv[i] = LDS_NOWHERE;
    }
#pragma unroll
    for (int s = -(WS > 2 * XS ? WS : 2 * XS); s < 0; ++s) {
      const int kw = s + WS, kx = s + 2 * XS - 1;   // (rows: of the steps kx and kx + 1)
      if (kw >= 0)
#pragma unroll
        for (int i = 0; i < WL; ++i) request_w(b, lds0, wave, lane * 16u, i, min(kw, n - 1), wring(RBL) + kw * WPLACE, kw < n);
      if ((s & 1) && kx >= 0)
#pragma unroll
        for (int i = 0; i < XL; ++i) request_x(b, p.xv, lds0, wave, i, min(kx, n - 2) >> 1, (kx >> 1) * xplace(RBL), kx < n);
    }
  }
  static __device__ __forceinline__ void first(const GemmStreamArgs& a, LdsPlaces& p, uint32_t xbytes, const LdsItem& it, const int* s_src, uint32_t lds0, int wave, int lane) {
    const int KT = a.KT;
    static_assert(LDS_NW % 2 == 0, "a wavefront's units are all of gate or all of up");
    p.w = (uint64_t)((NACC == 2 && (wave & 1) ? a.Wp2 : a.Wp) + (size_t)it.expert * a.expert_stride + (size_t)it.nt0 * KT * 64);
    p.wbytes = (uint32_t)it.tiles * (uint32_t)KT * 1024u;
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int t = wave + LDS_NW * i;
      const bool ok = t / NACC < it.tiles;
      p.wo[i] = (uint32_t)(ok ? t / NACC : 0) * (uint32_t)KT * 1024u;
      p.wv[i] = ok ? 0u : LDS_NOWHERE;
    }
    const LdsBuffers b(a, p, xbytes);
    if (it.rows <= 64) request_first<2>(a, p, b, it, s_src, lds0, wave, lane, KT);
    else if (it.rows <= 128) request_first<4>(a, p, b, it, s_src, lds0, wave, lane, KT);
    else if (it.rows <= 192) request_first<6>(a, p, b, it, s_src, lds0, wave, lane, KT);
    else request_first<8>(a, p, b, it, s_src, lds0, wave, lane, KT);
  }

  // All of K of one tile whose first stages are requested; `between` runs when the tile's operands are no longer needed, ahead of the stores.
  template <int RBL, typename F>
  static __device__ __forceinline__ void multiply(const GemmStreamArgs& a, const LdsPlaces& p, uint32_t xbytes, const LdsItem& it, uint8_t* smem, uint32_t lds0, const float* s_rs, const int* s_orow,
                                                  int wave, int lane, const F& between) {
    constexpr int XL = xl(RBL), XS = lds_xs(RBL), WS = lds_ws(RBL), NR = LDS_TW + RBL, NM = RBL * LDS_TW;
    constexpr uint32_t XP = xplace(RBL), WR0 = wring(RBL), WR1 = WR0 + WS * WPLACE;
    const int wr = wave % LDS_WR, wc = wave / LDS_WR, g = lane >> 4, f = lane & 15, n = a.KT;
    const uint32_t lane16 = lane * 16;
    const LdsBuffers b(a, p, xbytes);
    f32x4_t acc[RBL][LDS_TW];
#pragma unroll
    for (int rb = 0; rb < RBL; ++rb)
#pragma unroll
      for (int t = 0; t < LDS_TW; ++t) acc[rb][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t fx[2][RBL], fw[2][LDS_TW];
    // (row blocks go to the wavefronts in turn, so that those past the rows are shared out)
    const uint8_t* xb[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) xb[u] = smem + wr * 2048 + (ROWS ? (f >> 3) * 1024 + (f & 7) * 128 + ((4 * u + g) ^ (f & 7)) * 16 : u * 1024 + (int)lane16);
    const uint8_t* wb = smem + wc * LDS_TW * 1024 + lane16;
    auto read = [&](auto st_, auto qt, uint32_t xp, uint32_t wp) __attribute__((always_inline)) {   // operand q (weights first) of an even / odd step
      constexpr int S = decltype(st_)::value, q = decltype(qt)::value;
      if constexpr (q < LDS_TW) fw[S][q] = *(const u32x4_t*)(wb + wp + q * 1024);
      else fx[S][q - LDS_TW] = *(const u32x4_t*)(xb[S] + xp + LDS_WR * (q - LDS_TW) * 2048);
    };
    lds_wait_barrier<lds_behind(1, WS, XS, WL, XL)>();   // (stores of the tile before count too: then this waits for more)
    lds_each<0, NR>([&](auto q) __attribute__((always_inline)) { read(std::integral_constant<int, 0>{}, q, 0, WR0); });
    uint32_t xp = 0, xn = XS > 1 ? XP : 0, wp = WR0, wn = WR0 + WPLACE;   // places of this step's operands and of the next one's
    // A step's products, out of registers.  Between them the operands of step k + 1 have landed everywhere and nobody reads those of step k any more
    // (barrier): the reads of step k + 1, and the requests that take the places of what is done with.
    auto step = [&](auto st_, int k) __attribute__((always_inline)) {
      constexpr int S = decltype(st_)::value, PB = NM / 8, NQ = WL + (S ? XL : 0), NO = NQ + NR;
      const int kw = k + WS, kx = k + 2 * XS - 1;
      lds_each<0, NM>([&](auto i_) __attribute__((always_inline)) {
        constexpr int i = decltype(i_)::value, rb = i / LDS_TW, t = i % LDS_TW;
        acc[rb][t] = mfma_16x16x32<OPM_F16>(fw[S][t], fx[S][rb], acc[rb][t]);
        if constexpr (i == PB) {
          __builtin_amdgcn_sched_barrier(0);
          lds_wait_barrier<lds_behind(S, WS, XS, WL, XL)>();
        }
        if constexpr (i >= PB)
          lds_each<(i - PB) * NO / (NM - PB), (i - PB + 1) * NO / (NM - PB)>([&](auto j_) __attribute__((always_inline)) {
            constexpr int j = decltype(j_)::value, d0 = j * NQ / NO, d1 = (j + 1) * NQ / NO;
            if constexpr (d1 > d0) {
              if constexpr (d0 < WL) request_w(b, lds0, wave, lane16, d0, min(kw, n - 1), wp, kw < n);
              else request_x(b, p.xv, lds0, wave, d0 - WL, min(kx, n - 2) >> 1, xp, kx < n);
            } else read(std::integral_constant<int, 1 - S>{}, std::integral_constant<int, j - d0>{}, S ? xn : xp, wn);
          });
        __builtin_amdgcn_sched_barrier(0);
      });
      wp = wn;
      wn = wn + WPLACE == WR1 ? WR0 : wn + WPLACE;
      if (S) {
        xp = xn;
        xn = xn + XP == WR0 ? 0 : xn + XP;
      }
    };
    for (int k = 0; k < n; k += 2) {   // (an even number)
      step(std::integral_constant<int, 0>{}, k);
      step(std::integral_constant<int, 1>{}, k + 1);
    }
    lds_wait_barrier<0>();
    between();
#pragma unroll
    for (int rb = 0; rb < RBL; ++rb) {
      const int blk = wr + LDS_WR * rb, r = blk * 16 + f;
      if (blk * 16 >= it.rows) continue;   // uniform over the wavefront
      const float rs = s_rs[r];
      const int orow = s_orow[r];
#pragma unroll
      for (int t = 0; t < TWP; ++t)
        if (wc * TWP + t < it.tiles) gemm_epi_unit<EPI, !ROWS>(a, r < it.rows, orow, rs, it.nt0 + wc * TWP + t, g, acc[rb][t * NACC], acc[rb][t * NACC + NACC - 1], nullptr);
    }
  }
};

// cols: groups of features.  GATHER (gate / up): rows of X by token, the result in the experts' order, scaled by row_rs of the token; SCATTER (down): rows in
// the experts' order, the result to the (token, slot) row, scaled by its routing weight.
template <int EPI>
__global__ __launch_bounds__(LDS_THREADS, 2) void gemm_expert_kernel(const GemmStreamArgs a, const uint32_t xbytes, const int cols) {
  using T = LdsTile<EPI, true, true>;
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ float s_rs[2][256];
  __shared__ int s_orow[2][256], s_src[256];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // (opaque: what depends on the lane alone is otherwise computed for all row counts ahead of the choice)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), row = tid & 255;
  const int xcd = blockIdx.x & 7, wg = (int)blockIdx.x >> 3, wgs = (int)gridDim.x >> 3;
  const int list = xcd / a.tile_slices, slice = xcd % a.tile_slices, c0 = slice * cols / a.tile_slices, mine = (slice + 1) * cols / a.tile_slices - c0;   // (at least one: see gemm_expert_slices)
  const int items = (int)lds_uniform(a.n_tiles[list]) * mine, first_tile = list * a.tile_list;
  auto item = [&](int q, LdsItem& it) __attribute__((always_inline)) {
    const int j = q * wgs + (q & 1 ? wgs - 1 - wg : wg);
    if (j >= items) return false;
    const int t = first_tile + j / mine;
    it.m0 = (int)lds_uniform(a.tile_row0[t]); it.rows = (int)lds_uniform(a.tile_rows[t]); it.expert = (int)lds_uniform(a.tile_expert[t]); it.nt0 = (c0 + j % mine) * T::TPW; it.tiles = min(T::TPW, a.NT - it.nt0);
    return true;
  };
  auto sorted_of = [&](const LdsItem& it) __attribute__((always_inline)) { return a.sorted[it.m0 + min(row, it.rows - 1)]; };
  auto put_rows = [&](const LdsItem& it, int sv, int b, float& rs) __attribute__((always_inline)) {   // source and destination rows; the row's factor is requested
    if (EPI == SEPI_SWIGLU) {
      const int token = sv / a.top_k;
      if (tid < 256) { s_src[row] = token; s_orow[b][row] = it.m0 + row; }
      rs = a.row_rs[token];
    } else {
      if (tid < 256) { s_src[row] = it.m0 + min(row, it.rows - 1); s_orow[b][row] = sv; }
      rs = a.route_w[sv];
    }
  };
  LdsItem it;
  if (!item(0, it)) return;
  LdsPlaces p;
  {
    float rs;
    put_rows(it, sorted_of(it), 0, rs);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    T::first(a, p, xbytes, it, s_src, lds0, wave, lane);
    if (tid < 256) s_rs[0][row] = rs;
  }
  for (int q = 0;; ++q) {
    LdsItem nx;
    const bool more = item(q + 1, nx);
    int sv = 0;
    if (more) sv = sorted_of(nx);
    const int b = q & 1;
    float rs = 0.f;
    auto between = [&]() __attribute__((always_inline)) {   // the next tile's first stages, ahead of this one's stores
      if (!more) return;
      put_rows(nx, sv, b ^ 1, rs);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      T::first(a, p, xbytes, nx, s_src, lds0, wave, lane);
    };
    if (it.rows <= 64) T::template multiply<2>(a, p, xbytes, it, smem, lds0, s_rs[b], s_orow[b], wave, lane, between);
    else if (it.rows <= 128) T::template multiply<4>(a, p, xbytes, it, smem, lds0, s_rs[b], s_orow[b], wave, lane, between);
    else if (it.rows <= 192) T::template multiply<6>(a, p, xbytes, it, smem, lds0, s_rs[b], s_orow[b], wave, lane, between);
    else T::template multiply<8>(a, p, xbytes, it, smem, lds0, s_rs[b], s_orow[b], wave, lane, between);
    if (!more) break;
    if (tid < 256) s_rs[b ^ 1][row] = rs;   // (the K loop's barriers lie between this and its readers)
    it = nx;
  }
}

// The unembedding.  The row count is on the device.  XCD x has ranges of feature tiles x, x + 8, ..; the row tiles (of up to 256 rows, about alike) of a
// range sit next to each other on one XCD, so that its weights come in from memory once.  A workgroup's rows stay the same, its range is cut into groups of
// TPW tiles.  us per launch, gemm_mid.hip (up to 64 rows) or the tiled kernel / this one: 1.7B 17 rows 119 / 106, 35 130 / 114, 96 183 / 130, 512
// 501 / 380; 4B 64 191 / 150 (5.4 TB/s with what is stored), 128 209 / 171, 256 285 / 265; 8B 32 247 / 219, 256 444 / 424, 512 817 / 708.  Up to 16 rows
// the streaming kernel is the faster one (1.7B, 12 rows, 95 / 103).  From 256 rows on the matrix pipes at the board's power limit bound it: without its
// requests, 256 rows of 8B take 309 us, without its products 297, without its stores 347.  (X in rows, for models too small for fragment order: two or three registers a lane go to scratch;
// forwards of one layer, before this kernel / now: 512 columns, 151936 features, 64 rows 123 / 106, 512 350 / 297, 256 columns, 32000 features, 64 rows 96 / 89.)
template <bool ROWS, bool STREAM>
__global__ __launch_bounds__(LDS_THREADS, 2) void gemm_lds_kernel(const GemmStreamArgs a, const uint32_t xbytes) {
  using T = LdsTile<SEPI_STORE_F32, ROWS, STREAM>;
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ float s_rs[256];
  __shared__ int s_orow[256], s_src[256];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = (int)lds_uniform(*a.m_count), blocks = (M + 15) >> 4;
  if (M <= 0) return;
  const int xcd = blockIdx.x & 7, wg = (int)blockIdx.x >> 3, wgs = (int)gridDim.x >> 3;
  const int row_tiles = (blocks + 15) >> 4, per = (blocks + row_tiles - 1) / row_tiles, side = min(row_tiles, wgs), ranges = wgs / side;
  if (wg >= ranges * side) return;
  const int range = (wg / side) * 8 + xcd, nt_lo = (int)((long long)range * a.NT / (8 * ranges)), nt_hi = (int)((long long)(range + 1) * a.NT / (8 * ranges));
  if (nt_lo >= nt_hi) return;
  for (int rt = wg % side; rt * per < blocks; rt += side) {
    LdsItem it;
    it.m0 = rt * per * 16; it.rows = min(per * 16, M - it.m0); it.expert = 0; it.nt0 = nt_lo; it.tiles = min(T::TPW, nt_hi - nt_lo);
    // ---- the rows: sources and 1/rms from the producer's partial sums of squares ----
    {
      const int r = tid >> 1, sub = tid & 1, s = it.m0 + min(r, it.rows - 1), src = a.gather ? a.gather[s] : s;
      if (sub == 0) { s_src[r] = src; s_orow[r] = s; }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      LdsPlaces p;
      T::first(a, p, xbytes, it, s_src, lds0, wave, lane);
      const float v = lds_row_squares(a, src, sub);
      if (sub == 0) s_rs[r] = 1.0f / sqrtf(v / (float)a.K + a.eps);   // (read behind the K loop's barriers)
      for (;;) {
        LdsItem nx = it;
        nx.nt0 += T::TPW;
        nx.tiles = min(T::TPW, nt_hi - nx.nt0);
        const bool more = nx.tiles > 0;
        LdsPlaces np = p;
        auto between = [&]() __attribute__((always_inline)) {
          if (more) T::first(a, np, xbytes, nx, s_src, lds0, wave, lane);
        };
        if (it.rows <= 64) T::template multiply<2>(a, p, xbytes, it, smem, lds0, s_rs, s_orow, wave, lane, between);
        else if (it.rows <= 128) T::template multiply<4>(a, p, xbytes, it, smem, lds0, s_rs, s_orow, wave, lane, between);
        else if (it.rows <= 192) T::template multiply<6>(a, p, xbytes, it, smem, lds0, s_rs, s_orow, wave, lane, between);
        else T::template multiply<8>(a, p, xbytes, it, smem, lds0, s_rs, s_orow, wave, lane, between);
        if (!more) break;
        it = nx;
        p = np;
      }
    }
    __syncthreads();   // the next rows take the same LDS
  }
}

// ---- gate / up of many rows ----
// Tiles of 64 RBW rows x 192 features (96 of gate and up each): with eight wavefronts 4 x 2, each RBW row blocks x 6 feature tiles, a step of 32 columns takes
// 0.58 KB of lines per product where the 128 x 128 pairs of the tiled kernel take 0.75, and the chip is filled without sharing K.  Both operands in fragment order,
// five to eight stages of 32 columns.  The row count is on the device: P row tiles expected, whose height follows it.
constexpr int LDS_GU_WR = 4, LDS_GU_WC = 2, LDS_GU_TW = 6, LDS_GU_TA = LDS_GU_WC * LDS_GU_TW, LDS_GU_TPW = LDS_GU_TA / 2;   // (TPW: pairs of a workgroup)
constexpr int lds_gu_stages(int RBW) { return RBW == 4 ? 5 : RBW == 3 ? 6 : RBW == 2 ? 7 : 8; }
constexpr int lds_gu_stage(int RBW) { return (LDS_GU_WR * RBW + LDS_GU_TA) * 1024; }
constexpr int LDS_GU_DUMP = 144 * 1024;   // where units that do not exist go
static_assert(5 * lds_gu_stage(4) <= LDS_GU_DUMP && 6 * lds_gu_stage(3) <= LDS_GU_DUMP && 7 * lds_gu_stage(2) <= LDS_GU_DUMP && 8 * lds_gu_stage(1) <= LDS_GU_DUMP, "LDS");

template <int RBW>
__device__ __forceinline__ void lds_gateup_body(const GemmStreamArgs& a, const int groups, const int P, const int M, const uint32_t xbytes, uint8_t* smem, float* s_rs) {
  constexpr int NW = LDS_NW, WR = LDS_GU_WR, TW = LDS_GU_TW, TPW = LDS_GU_TPW, RB = WR * RBW, XU = RB, WU = LDS_GU_TA;
  constexpr int XL = (XU + NW - 1) / NW, WL = (WU + NW - 1) / NW, L = XL + WL, ST = lds_gu_stages(RBW), NR = RBW + TW, NM = RBW * TW;
  constexpr uint32_t STAGE = lds_gu_stage(RBW);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)smem;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));   // (opaque: what depends on the lane alone is otherwise computed for all heights ahead of the choice)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave % WR, wc = wave / WR, g = lane >> 4, f = lane & 15;
  const int KT = a.KT, blocks = (M + 15) >> 4, tiles = min(P, (blocks + RB - 1) / RB);
  // XCD i % 8 has the groups of features c % 8 == i % 8, all row tiles of one next to each other: its weights come in from memory once
  const int s_ = (int)blockIdx.x >> 3, grp = (s_ / tiles) * 8 + (blockIdx.x & 7);
  if (grp >= groups) return;
  const uint32_t wbytes = (uint32_t)min(TPW, a.NT - grp * TPW) * (uint32_t)KT * 1024u;
  // (a wavefront requests units of gate or of up only)
  const uint64_t matrix = (uint64_t)((wave & 1 ? a.Wp2 : a.Wp) + (size_t)grp * TPW * KT * 64);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)lds_uniform((uint32_t)(matrix >> 32)) << 32 | lds_uniform((uint32_t)matrix)), 0, wbytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)a.X, 0, xbytes, 0x00020000);
  const uint32_t lane16 = lane * 16;
  uint32_t wo[WL], wv[WL], xo[XL], xv[XL];
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int t = wave + NW * i;
    const bool ok = t < WU && grp * TPW + (t >> 1) < a.NT;
    wo[i] = (ok ? (uint32_t)(t >> 1) : 0u) * (uint32_t)KT * 1024u;
    wv[i] = ok ? 0u : LDS_NOWHERE;
  }
  auto request = [&](auto i_, int k, uint32_t buf) __attribute__((always_inline)) {   // weights first
    constexpr int i = decltype(i_)::value;
    const uint32_t ko = (uint32_t)min(k, KT - 1) * 1024u, lanes = k < KT ? lane16 : LDS_NOWHERE;
    if constexpr (i < WL) {
      const int t = wave + NW * i;
      lds_request<false>(rw, lanes | wv[i], wo[i] + ko, lds0 + (WU % NW == 0 || t < WU ? buf + (XU + t) * 1024u : LDS_GU_DUMP));
    } else {
      const int t = wave + NW * (i - WL);
      lds_request<false>(rx, lanes | xv[i - WL], xo[i - WL] + ko, lds0 + (XU % NW == 0 || t < XU ? buf + t * 1024u : LDS_GU_DUMP));
    }
  };
  for (int pass = s_ % tiles; pass * RB < blocks; pass += tiles) {
    const int m0 = pass * RB * 16, Mloc = min(RB * 16, M - m0);
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int t = wave + NW * i;
      const bool ok = t < XU && t * 16 < Mloc;
      xo[i] = (uint32_t)((m0 >> 4) + (ok ? t : 0)) * (uint32_t)KT * 1024u;
      xv[i] = ok ? 0u : LDS_NOWHERE;
    }
    lds_each<0, ST>([&](auto s) __attribute__((always_inline)) {
      lds_each<0, L>([&](auto i) __attribute__((always_inline)) { request(i, decltype(s)::value, decltype(s)::value * STAGE); });
    });
    {   // 1/rms of the rows from the producer's partial sums of squares
      const int r = tid >> 1, sub = tid & 1;
      const float v = lds_row_squares(a, min(m0 + r, M - 1), sub);
      if (r < RB * 16 && sub == 0) s_rs[r] = 1.0f / sqrtf(v / (float)a.K + a.eps);
    }
    f32x4_t acc[RBW][TW];
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb)
#pragma unroll
      for (int t = 0; t < TW; ++t) acc[rb][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t fx[2][RBW], fw[2][TW];
    const uint8_t* xb = smem + wr * 1024 + lane16;   // (row blocks go to the wavefronts in turn)
    const uint8_t* wb = smem + (XU + wc * TW) * 1024 + lane16;
    auto read = [&](auto st_, auto j_, uint32_t buf) __attribute__((always_inline)) {
      constexpr int S = decltype(st_)::value, j = decltype(j_)::value;
      if constexpr (j < TW) fw[S][j] = *(const u32x4_t*)(wb + buf + j * 1024);
      else fx[S][j - TW] = *(const u32x4_t*)(xb + buf + WR * (j - TW) * 1024);
    };
    lds_wait_barrier<L * (ST - 1)>();
    lds_each<0, NR>([&](auto j) __attribute__((always_inline)) { read(std::integral_constant<int, 0>{}, j, 0); });
    uint32_t buf = 0, nbuf = STAGE;
    // (as in multiply() above: stage k + 1 lands, the reads of it and the requests of stage k + ST between the products of stage k)
    auto step = [&](auto st_, int k) __attribute__((always_inline)) {
      constexpr int S = decltype(st_)::value, PB = NM / 8, NO = L + NR;
      lds_each<0, NM>([&](auto i_) __attribute__((always_inline)) {
        constexpr int i = decltype(i_)::value, rb = i / TW, t = i % TW;
        acc[rb][t] = mfma_16x16x32<OPM_F16>(fw[S][t], fx[S][rb], acc[rb][t]);
        if constexpr (i == PB) {
          __builtin_amdgcn_sched_barrier(0);
          lds_wait_barrier<L * (ST - 2)>();
        }
        if constexpr (i >= PB)
          lds_each<(i - PB) * NO / (NM - PB), (i - PB + 1) * NO / (NM - PB)>([&](auto j_) __attribute__((always_inline)) {
            constexpr int j = decltype(j_)::value, d0 = j * L / NO, d1 = (j + 1) * L / NO;
            if constexpr (d1 > d0) request(std::integral_constant<int, d0>{}, k + ST, buf);
            else read(std::integral_constant<int, 1 - S>{}, std::integral_constant<int, j - d0>{}, nbuf);
          });
        __builtin_amdgcn_sched_barrier(0);
      });
      buf = nbuf;
      nbuf = nbuf + STAGE == ST * STAGE ? 0 : nbuf + STAGE;
    };
    for (int k = 0; k < KT; k += 2) {   // (an even number)
      step(std::integral_constant<int, 0>{}, k);
      step(std::integral_constant<int, 1>{}, k + 1);
    }
    lds_wait_barrier<0>();
#pragma unroll
    for (int rb = 0; rb < RBW; ++rb) {
      const int blk = wr + WR * rb, r = blk * 16 + f;
      if (blk * 16 >= Mloc) continue;   // uniform over the wavefront
      const float rs = s_rs[r];
#pragma unroll
      for (int t = 0; t < TW / 2; ++t)
        gemm_epi_unit<SEPI_SWIGLU, true>(a, r < Mloc, m0 + min(r, Mloc - 1), rs, grp * TPW + wc * (TW / 2) + t, g, acc[rb][2 * t], acc[rb][2 * t + 1], nullptr);
    }
    __syncthreads();   // rows beyond the expected ones take the same LDS
  }
}

__global__ __launch_bounds__(LDS_THREADS, 2) void gemm_lds_gateup_kernel(const GemmStreamArgs a, const int P, const int groups, const uint32_t xbytes) {
  extern __shared__ __align__(16) uint8_t smem[];
  __shared__ float s_rs[256];
  const int M = (int)lds_uniform(*a.m_count), blocks = (M + 15) >> 4;
  if (M <= 0) return;
  const int rbw = ((blocks + P - 1) / P + LDS_GU_WR - 1) / LDS_GU_WR;   // heights by the rows there are
  if (rbw <= 1) lds_gateup_body<1>(a, groups, P, M, xbytes, smem, s_rs);
  else if (rbw == 2) lds_gateup_body<2>(a, groups, P, M, xbytes, smem, s_rs);
  else if (rbw == 3) lds_gateup_body<3>(a, groups, P, M, xbytes, smem, s_rs);
  else lds_gateup_body<4>(a, groups, P, M, xbytes, smem, s_rs);
}

// Row tiles and time of a launch: rounds of workgroups, each KT steps and its ends (fitted with KT 64, 80 and 128, one round and two).
// How far the choice between this kernel, the tiled one and the blocks is from the fastest of them, us per layer on average over 128 to 1024 rows
// in steps of 64, in brackets without this kernel: 4096 x 12288 0.8 (18), 2560 x 9728 1.1 (8), 2048 x 11008 0.6 (11), 2048 x 6144 0.2 (8), 3072 x 8192 0.9 (3).
// Matrices of less than 48 MB together, or of less than 2048 columns, are given to it where it is 1.15 times faster than the others by the estimates:
// of 255 forwards of four layers (17 matrices from 512 x 8192 to 4096 x 2048, 128 to 1536 rows) it then has 48, of which the least improved takes 0.99 of the time
// without it, the most 0.88; by the bare estimates it has 93, and ten of them take 1.02 to 1.03 times as long.
struct LdsGateup { int P; double us; };
static LdsGateup lds_gateup(const GemmStreamArgs& a) {
  constexpr double per_kt[5] = {0, 0, .44, .58, .65}, ends[5] = {0, 0, 6.0, 8.0, 11.0};
  LdsGateup best{0, 1e30};
  const int groups = (a.NT + LDS_GU_TPW - 1) / LDS_GU_TPW;
  for (int rbw = 2; rbw <= 4; ++rbw) {
    const int P = (a.m_hint + 64 * rbw - 1) / (64 * rbw);
    const double us = std::ceil((groups + 7) / 8 * P / (a.coop_wgs / 8.0)) * (a.KT * per_kt[rbw] + ends[rbw]);
    if (us < best.us) best = {P, us};
  }
  return best;
}
double gemm_lds_gateup_us(const GemmStreamArgs& a) {
  if (a.KT < 24 || (long long)a.NT * a.KT < 8192) return 1e30;   // (matrices of less than 16 MB together, or of less than 768 columns: little to gain, 2048 x 2048 0.2 us a layer)
  if (a.x_lo != LO_F16P || a.coop_wgs < 8 || a.KT % 2 || a.grouped != GROUP_NONE || (long long)((a.x_rows + 15) / 16) * a.KT * 1024 >= 0xfffff000LL) return 1e30;
  return lds_gateup(a).us * (a.KT < 64 || (long long)a.NT * a.KT < 24576 ? 1.15 : 1.0);   // (see lds_gateup)
}

// The unembedding: half operands, whole steps of 64 columns, 32-bit offsets into the rows, and enough feature tiles for each of the kernel's ranges.  A workgroup's K loop
// takes as long for one feature tile as for 16, so a small vocabulary wants the kernels that cut K or take fewer features a workgroup (mid-size, streaming, tiled).  us per launch, this
// kernel / the one that the others' rules pick, as the difference, at 2048 columns: 8192 features (2 tiles a range of one row tile) 32 rows +9, 64 +7, 128 -12, 256 +17, 512 +14; 16384 +3,
// -3, -6, +14, +8; 24576 +2, -3, -1, +11, -15; 36864 +1, -7, 0, -16, -16; 50304 -17, -19, -3, -26, -38; at 4096 columns 8192 features +14, +11, +12, +41, +20; 24576 +3, -14,
// -17, -9, -21; at 1024 columns 8192 features +7, +6, -6, +3, +4.  257 to 384 rows with 17 to 20 tiles a range (the second group of 16 nearly empty), 4096 columns +18 to +26.  Over 780 such cases
// (512 to 8192 columns, 2048 to 65536 features, 17 to 1024 rows) the rule is 0.3 us from the faster one on average; this kernel everywhere 4.2, nowhere 15.
bool gemm_lds_takes(int kind, const GemmStreamArgs& a) {
  if ((a.x_lo != LO_F16 && a.x_lo != LO_F16P) || a.coop_wgs < 1 || a.KT % 2 || a.grouped != GROUP_NONE || (long long)((a.x_rows + 15) / 16) * a.KT * 1024 >= 0xfffff000LL) return false;
  if (kind != SEPI_STORE_F32 || !a.gather || a.m_hint <= 16) return false;
  const int rows = a.m_hint, row_tiles = (rows + 255) / 256, wgs = std::max(1, a.coop_wgs / 8);
  const double per = a.NT / (8.0 * (wgs / std::min(row_tiles, wgs)));   // feature tiles of a range
  if (rows > 256 && rows <= 384 && per > 16.0 && per < 21.0) return false;
  const int least = rows <= 32 ? 7 : rows <= 64 && a.x_lo == LO_F16P ? 6 : rows <= 128 ? std::min(a.KT / 32, 4) : rows <= 192 && a.KT <= 32 ? 0 : rows <= 256 && a.KT >= 128 ? 5 : 9;
  return per >= least;
}
static void lds_attribute(const void* fn, unsigned bytes, bool (&done)[64]) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
  if (!done[dev] && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess) done[dev] = true;   // on failure the launch fails too, and the entry point reports that error
}
template <bool ROWS, bool STREAM>
static void launch_lds(hipStream_t st, const GemmStreamArgs& a, uint32_t xbytes) {
  static bool lds_set[64];
  lds_attribute((const void*)gemm_lds_kernel<ROWS, STREAM>, LDS_BYTES, lds_set);
  S2D2_LAUNCH((gemm_lds_kernel<ROWS, STREAM>), dim3(std::max(1, a.coop_wgs / 8) * 8), dim3(LDS_THREADS), LDS_BYTES, st, a, xbytes);
}
void launch_gemm_lds(hipStream_t st, int kind, const GemmStreamArgs& a) {
  const uint32_t xbytes = (uint32_t)((a.x_rows + 15) / 16) * (uint32_t)a.KT * 1024u;   // (in rows: at least as many)
  if (kind == SEPI_SWIGLU) {
    static bool lds_set[64];
    lds_attribute((const void*)gemm_lds_gateup_kernel, LDS_GU_DUMP + 1024, lds_set);
    const int P = lds_gateup(a).P, groups = (a.NT + LDS_GU_TPW - 1) / LDS_GU_TPW;
    S2D2_LAUNCH(gemm_lds_gateup_kernel, dim3((groups + 7) / 8 * 8 * P), dim3(LDS_THREADS), LDS_GU_DUMP + 1024, st, a, P, groups, xbytes);
    return;
  }
  const bool rows = a.x_lo == LO_F16, stream = a.m_hint <= 256;   // stream: one row tile, every weight is requested once
  if (rows && stream) launch_lds<true, true>(st, a, xbytes);
  else if (rows) launch_lds<true, false>(st, a, xbytes);
  else if (stream) launch_lds<false, true>(st, a, xbytes);
  else launch_lds<false, false>(st, a, xbytes);
}

template <int EPI>
static void launch_expert(hipStream_t st, const GemmStreamArgs& a, uint32_t xbytes) {
  static bool lds_set[64];
  lds_attribute((const void*)gemm_expert_kernel<EPI>, LDS_BYTES, lds_set);
  const int wgs = std::max(1, a.coop_wgs / 8) * 8;
  S2D2_LAUNCH((gemm_expert_kernel<EPI>), dim3(wgs), dim3(LDS_THREADS), LDS_BYTES, st, a, xbytes, (a.NT + LdsTile<EPI, true, true>::TPW - 1) / LdsTile<EPI, true, true>::TPW);
}

static int expert_groups(int features, int per) { return (features / 16 + per - 1) / per; }   // of features, a workgroup's tile each
// Half operands in rows, whole stages of 64 columns, 32-bit offsets.  Few experts of small matrices and many rows: tiles of 256 x 256 leave most compute units
// without one.  Drafts of two layers, us, tiled kernel / this one: 2 experts of 2048 x 2048, both chosen, 128 rows 294 / 305, 256 316 / 383, 512 357 / 418; 8 of 1024 x 1024, 2 chosen, 512 rows
// 292 / 317, 1024 349 / 369; but 8 of 2048 x 2048 256 rows 364 / 362, 1024 527 / 485, and few rows of 2 experts 229 / 217, of 8 195 / 182.  (Where the two are
// close the tiled kernel is ahead here and there: 32 of 1024 x 1024, 4 chosen, 512 rows 313 / 331, 4 of 2048 x 4096, 1 chosen, up to 8 rows 239 / 248.)
bool gemm_expert_takes(int experts, int d_model, int d_expert, int rows, int rows_expected, int top_k, int x_lo, int cus) {
  const long long most = std::max((long long)rows * d_model, (long long)rows * top_k * d_expert) * 2;
  if (experts * expert_groups(d_expert, LdsTile<SEPI_SWIGLU, true, true>::TPW) * 2 < cus && rows_expected * top_k >= 64 * experts) return false;
  return x_lo == LO_F16 && d_model % 64 == 0 && d_expert % 64 == 0 && most < 0xfffff000LL && (long long)((d_expert + 15) / 16) * d_model * 32 < 0xfffff000LL;
}
// Slices of the features that the XCDs of a list have between them.  Of few experts, or of the two that one row chooses, whole ones leave XCDs with nothing
// to do or with twice as much as others.  Drafts of two layers, us, tiled kernel / one slice / four: 4 experts of 4096 x 8192, 2 chosen, 1 row 448 / 518 / 413, 1024 rows 1479 / 2498 / 1275;
// 8 of 4096 x 14336 1 row 611 / 841 / 582, 512 rows 1722 / 2009 / 1637; 8 of 2048 x 4096 1024 rows 664 / 852 / 650; 12 of 2048 x 1408 482 / 549 / 458.  16 experts and more by the
// expert: its rows are read on one XCD (64 of 2048 x 1024, four layers, 9 rows 549 / 543, 256 rows 1036 / 1041, verification of 144 rows 844 / 867).
int gemm_expert_slices(int experts, int d_model, int d_expert) {
  const int groups = std::min(expert_groups(d_expert, LdsTile<SEPI_SWIGLU, true, true>::TPW), expert_groups(d_model, LdsTile<SEPI_STORE_F32, true, true>::TPW));
  int s = experts < 16 ? 4 : 1;
  while (s > groups) s >>= 1;
  return s;
}
void launch_gemm_expert(hipStream_t st, int kind, const GemmStreamArgs& a, int x_rows) {
  const uint32_t xbytes = (uint32_t)x_rows * (uint32_t)a.ldx * 2u;
  if (kind == SEPI_SWIGLU) launch_expert<SEPI_SWIGLU>(st, a, xbytes);
  else launch_expert<SEPI_STORE_F32>(st, a, xbytes);
}

}  // namespace s2d2
