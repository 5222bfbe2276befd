// Epilogue of the packed-weight GEMMs on one 16 x 16 accumulator in MFMA register order, shared by the tiled, the
// mid-size and the block kernels and those through LDS.
#pragma once
#include "s2d2_internal.h"

namespace s2d2 {

// v0 (and v1, the up projection, for SwiGLU): v[i] = sum of output row orow (this lane's row; live: it exists), feature
// nt * 16 + 4 g + i, g = lane / 16; rs scales it.  The whole wavefront calls it with one nt (the norm's partial sums and
// the rotation pairs travel between lanes); nt >= NT does nothing.  h0 (SEPI_ADD_F32): the residual's four values at that
// place where the caller has requested them ahead of time, else they are read here; sq_sum: takes the row's sum of squares
// instead of the tile's entry in ss_out; ahead: what gemm_epi_request has read for this place (and the sequence of the row and
// its first row, for the values' copy), else read here.  FRAG_OUT: activation rows may be
// wanted in fragment order; false where they never are.  (Both keep instructions out of the tiled kernel, whose unsplit
// epilogue is unrolled over all units of a tile: values read in a region of their own and the layout chosen at run time
// made its residual-add kernel 18653 instructions for 16873.)
struct EpiAhead { float4 a, b; int seq, row0; };   // see gemm_epi_request
template <int EPI, bool FRAG_OUT>
__device__ __forceinline__ void gemm_epi_unit(const GemmStreamArgs& a, const bool live, const int orow, const float rs,
                                              const int nt, const int g, const f32x4_t& v0, const f32x4_t& v1, const float4* h0, float* sq_sum = nullptr,
                                              const EpiAhead* ahead = nullptr) {
  if (nt >= a.NT) return;   // uniform over the wavefront
  const int n = nt * 16 + 4 * g;
  auto put4 = [&](bf16_t* base, int lo, int ld, float x, float y, float z, float w) __attribute__((always_inline)) {
    if (FRAG_OUT) act_put4(base, lo, orow, n, ld, x, y, z, w);
    else act_store4(base + (size_t)orow * ld + n, lo, x, y, z, w);
  };
  if (EPI == SEPI_STORE_F32) {
    if (live) {
      float* op = (float*)a.out + (size_t)orow * a.ldo + n;
      const f32x4_t v = v0 * rs;
      if (n + 3 < a.N) *(float4*)op = make_float4(v[0], v[1], v[2], v[3]);
      else
        for (int i = 0; i < 4; ++i)
          if (n + i < a.N) op[i] = v[i];
    }
  } else if (EPI == SEPI_ADD_F32) {   // N is a multiple of 16 here: four features per lane as one 16-byte access
    float hv[4] = {0.f, 0.f, 0.f, 0.f};
    if (live) {
      float4* hp = (float4*)((float*)a.out + (size_t)orow * a.ldo + n);
      const float4 h = h0 ? *h0 : *hp;
      hv[0] = h.x + v0[0] * rs;
      hv[1] = h.y + v0[1] * rs;
      hv[2] = h.z + v0[2] * rs;
      hv[3] = h.w + v0[3] * rs;
      *hp = make_float4(hv[0], hv[1], hv[2], hv[3]);
      if (a.xg_out) {
        const float4 gn = ahead ? ahead->a : *(const float4*)(a.gain_next + n);
        put4(a.xg_out, a.xg_lo, a.xg_ld, hv[0] * gn.x, hv[1] * gn.y, hv[2] * gn.z, hv[3] * gn.w);
      }
    }
    if (a.ss_out) {
      float sq = (hv[0] * hv[0] + hv[1] * hv[1]) + (hv[2] * hv[2] + hv[3] * hv[3]);
      sq += __shfl_xor(sq, 16, 64);
      sq += __shfl_xor(sq, 32, 64);
      if (sq_sum) *sq_sum += sq;
      else if (live && g == 0) a.ss_out[(size_t)orow * a.ss_stride + nt] = sq;
    }
  } else if (EPI == SEPI_SWIGLU) {
    if (live) {
      float sv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float gate = v0[i] * rs, up = v1[i] * rs;
        sv[i] = gate / (1.0f + __expf(-gate)) * up;
      }
      put4((bf16_t*)a.out, a.out_lo, a.ldo, sv[0], sv[1], sv[2], sv[3]);
    }
  } else {  // SEPI_QKV_ROPE: features 0-7 of a tile pair with features 8-15 (lanes 32 apart)
    const int D = a.D, half = D >> 1, tiles_per_head = D / 16;
    const int head = nt / tiles_per_head, i0 = 8 * (nt % tiles_per_head) + 4 * (g & 1);
    float own[4], oth[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      own[i] = v0[i] * rs;
      oth[i] = __shfl_xor(own[i], 32, 64);
    }
    if (live) {
      const bool second = g >= 2;   // this lane holds x2 (element i + D/2) of the pair
      if (head < a.Hq + a.Hkv) {
        const bool is_q = head < a.Hq;
        bf16_t* dst = is_q ? a.q_out + (size_t)orow * a.q_ld + head * D
                           : a.k_out + ((size_t)orow * a.Hkv + (head - a.Hq)) * D;
        const float4 c01 = ahead ? ahead->a : *(const float4*)(a.rope_cs + (size_t)orow * half + i0), c23 = ahead ? ahead->b : *(const float4*)(a.rope_cs + (size_t)orow * half + i0 + 2);
        const float cs_c[4] = {c01.x, c01.z, c23.x, c23.z}, cs_s[4] = {c01.y, c01.w, c23.y, c23.w};
        float y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = second ? own[i] * cs_c[i] + oth[i] * cs_s[i] : own[i] * cs_c[i] - oth[i] * cs_s[i];
        // queries in the storage the attention kernel reads (q_lo); keys always as one bf16 plane (the cache's type)
        act_store4(dst + i0 + (second ? half : 0), is_q ? a.q_lo : 0, y[0], y[1], y[2], y[3]);
        if (!is_q && a.k16_out)   // the window's keys once more as half values (the attention kernel's copy)
          act_store4(a.k16_out + ((size_t)orow * a.Hkv + (head - a.Hq)) * D + i0 + (second ? half : 0), LO_F16, y[0], y[1], y[2], y[3]);
      } else {
        const int vh = head - a.Hq - a.Hkv;
        bf16_t* dst = a.v_out + ((size_t)orow * a.Hkv + vh) * D + (second ? half : 0);
        const int sq = ahead ? ahead->seq : a.row_seq[orow], tw = orow - (ahead ? ahead->row0 : a.seq_row0[sq]);
        bf16_t b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = f32_to_bf16(own[i]);
        *(uint2*)(dst + i0) = make_uint2((uint32_t)b[0] | ((uint32_t)b[1] << 16), (uint32_t)b[2] | ((uint32_t)b[3] << 16));
        if (a.vT_out) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            a.vT_out[((size_t)(sq * a.Hkv + vh) * D + i0 + i + (second ? half : 0)) * a.wpad + tw] = a.win_f16 ? f32_to_f16_bits(own[i]) : b[i];
        }
      }
    }
  }
}

// What gemm_epi_unit reads besides the residual, requested ahead of time for all units of a wavefront: unit by unit, between the stores,
// each read is waited for (rotation epilogue, 8B shape, 256 / 512 rows: 6 and 9 us of 32 and 52).
template <int EPI>
__device__ __forceinline__ void gemm_epi_request(const GemmStreamArgs& a, const int orow, const int nt, const int g, EpiAhead& e) {
  e.a = e.b = make_float4(0.f, 0.f, 0.f, 0.f);
  if (EPI == SEPI_ADD_F32 && a.xg_out) e.a = *(const float4*)(a.gain_next + nt * 16 + 4 * g);
  if (EPI == SEPI_QKV_ROPE) {   // (places without a rotation read one all the same)
    const float4* cs = (const float4*)(a.rope_cs + (size_t)orow * (a.D >> 1) + 8 * (nt % (a.D / 16)) + 4 * (g & 1));
    e.a = cs[0];
    e.b = cs[1];
  }
}

}  // namespace s2d2
