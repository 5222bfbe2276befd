// Y[m, n] = sum_k X[m, k] * W[n, k] on MFMA, fp32 accumulation.
//
// Weight-streaming kernel for the decode regime (a handful of window rows against a large
// weight matrix): the arithmetic intensity is ~M flop per weight byte, so the kernel is bound by
// reading W once from HBM.  One workgroup owns 16 output features and 16 rows; its four
// wavefronts split K and each lane streams 16-byte pieces of "its" weight row straight from
// global memory into the MFMA A operand (no LDS on the weight path), the rows of X (tiny,
// L2-resident) are the B operand.  Partial sums of the four waves are combined through LDS in
// a fixed order, so results are deterministic.  Larger M is covered by more row tiles.
#include "s2d2_internal.h"
#include "../../include/s2d2.h"

namespace s2d2 {

template <typename T> struct Mma;

template <> struct Mma<bf16_t> {
  static constexpr int KV = 8;  // elements per 16-byte fragment
  __device__ static __forceinline__ f32x4_t run(const uint4& a, const uint4& b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
  }
};

template <> struct Mma<float> {
  static constexpr int KV = 4;
  __device__ static __forceinline__ f32x4_t run(const uint4& a, const uint4& b, f32x4_t c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    return c;
  }
};

template <typename T, int EPI, int PASSES>
__global__ __launch_bounds__(256) void gemm_rows16_kernel(const T* __restrict__ X, int ldx,
                                                          const T* __restrict__ W, int K, int N,
                                                          const int32_t* __restrict__ m_count,
                                                          void* __restrict__ out, int ldo) {
  constexpr int KV = Mma<T>::KV;
  constexpr int KSTEP = 4 * KV;      // k covered by one fragment load of the whole wave
  constexpr int U = 4;               // fragment loads in flight per operand
  constexpr int KC = U * KSTEP;
  constexpr int NACC = EPI == EPI_SWIGLU ? 2 : 1;
  __shared__ float red[4][NACC][256];

  const int M = *m_count;
  const int m0 = blockIdx.y * 16;
  if (m0 >= M) return;
  const int n0 = blockIdx.x * 16;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (scalar: the K tests below are then scalar branches)
  const int g = lane >> 4, f = lane & 15;

  const int wn = min(n0 + f, N - 1);
  const bool row_ok = (m0 + f) < M;
  const T* wp = W + (size_t)wn * K + g * KV;
  const T* wp2 = wp + (size_t)N * K;  // up projection (SwiGLU only)
  const T* xp = X + (size_t)(row_ok ? m0 + f : m0) * ldx + g * KV;

  f32x4_t acc[NACC];
  for (int a = 0; a < NACC; ++a) acc[a] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  for (int k0 = wave * KC; k0 < K; k0 += PASSES * 4 * KC) {
    constexpr int UP = U * PASSES;
    uint4 wa[UP], wb[UP], xb[UP];
    auto k_of = [&](int t) { return k0 + t / U * (4 * KC) + t % U * KSTEP; };
#pragma unroll
    for (int t = 0; t < UP; ++t) {
      // unconditional loads, clamped to K (a multiple of KSTEP): under a condition they would wait for each other;
      // window rows past the count read row m0, their results are never stored
      const int k = min(k_of(t), K - KSTEP);
      wa[t] = *(const uint4*)(wp + k);
      if (EPI == EPI_SWIGLU) wb[t] = *(const uint4*)(wp2 + k);
      xb[t] = *(const uint4*)(xp + k);
    }
    auto mac = [&](int t) __attribute__((always_inline)) {
      acc[0] = Mma<T>::run(wa[t], xb[t], acc[0]);
      if (EPI == EPI_SWIGLU) acc[NACC - 1] = Mma<T>::run(wb[t], xb[t], acc[NACC - 1]);
    };
    if (k_of(UP - 1) + KSTEP <= K) {   // whole passes: nothing between their loads and their products
#pragma unroll
      for (int t = 0; t < UP; ++t) mac(t);
    } else {
#pragma unroll
      for (int t = 0; t < UP; ++t)
        if (k_of(t) < K) mac(t);
    }
  }
  // acc[a][i] = Y[m0 + f][n0 + 4 g + i]
  for (int a = 0; a < NACC; ++a)
    for (int i = 0; i < 4; ++i) red[wave][a][i * 64 + lane] = acc[a][i];
  __syncthreads();
  const int row = threadIdx.x >> 4, fe = threadIdx.x & 15;
  const int src = (fe & 3) * 64 + (fe >> 2) * 16 + row;
  float v[NACC];
  for (int a = 0; a < NACC; ++a) v[a] = (red[0][a][src] + red[1][a][src]) + (red[2][a][src] + red[3][a][src]);
  const int m = m0 + row, n = n0 + fe;
  if (m >= M || n >= N) return;
  if (EPI == EPI_STORE_F32) {
    ((float*)out)[(size_t)m * ldo + n] = v[0];
  } else if (EPI == EPI_ADD_F32) {
    ((float*)out)[(size_t)m * ldo + n] += v[0];
  } else {
    const float gate = v[0], up = v[NACC - 1];
    ((T*)out)[(size_t)m * ldo + n] = from_f32<T>(gate / (1.0f + __expf(-gate)) * up);
  }
}

template <typename T, int EPI>
static void launch_e(hipStream_t st, const T* X, int ldx, const T* W, int K, int N, const int32_t* m_count, int m_cap, void* out, int ldo) {
  const dim3 grid((N + 15) / 16, (m_cap + 15) / 16);
  // A pass of the four wavefronts covers 16 fragments (256 inputs in fp32).  Where K is longer and the workgroups are at
  // most one per compute unit, the loads of up to four passes are in flight at once (down projection of the fp32 model, 16
  // workgroups, K 768: 4.8 us per launch, 10 one pass at a time); past that the registers are better spent on further
  // workgroups.  The products keep their order, so a row's result does not depend on the form.
  const int passes = (K + 16 * 4 * Mma<T>::KV - 1) / (16 * 4 * Mma<T>::KV);
#define S2D2_ROWS16(P) S2D2_LAUNCH((gemm_rows16_kernel<T, EPI, P>), grid, dim3(256), 0, st, X, ldx, W, K, N, m_count, out, ldo)
  if (passes == 1 || (long long)grid.x * grid.y > 256) S2D2_ROWS16(1);
  else if (passes == 2) S2D2_ROWS16(2);
  else if (passes == 3) S2D2_ROWS16(3);
  else S2D2_ROWS16(4);
#undef S2D2_ROWS16
}

template <typename T>
static void launch_t(hipStream_t st, GemmEpilogue epi, const T* X, int ldx, const T* W, int K, int N,
                     const int32_t* m_count, int m_cap, void* out, int ldo) {
  switch (epi) {
    case EPI_STORE_F32: launch_e<T, EPI_STORE_F32>(st, X, ldx, W, K, N, m_count, m_cap, out, ldo); break;
    case EPI_ADD_F32: launch_e<T, EPI_ADD_F32>(st, X, ldx, W, K, N, m_count, m_cap, out, ldo); break;
    case EPI_SWIGLU: launch_e<T, EPI_SWIGLU>(st, X, ldx, W, K, N, m_count, m_cap, out, ldo); break;
  }
}

void launch_gemm(hipStream_t st, int dtype, GemmEpilogue epi, const void* X, int ldx, const void* W, int K,
                 int N, const int32_t* m_count, int m_cap, void* out, int ldo) {
  if (dtype == S2D2_BF16)
    launch_t<bf16_t>(st, epi, (const bf16_t*)X, ldx, (const bf16_t*)W, K, N, m_count, m_cap, out, ldo);
  else
    launch_t<float>(st, epi, (const float*)X, ldx, (const float*)W, K, N, m_count, m_cap, out, ldo);
}

}  // namespace s2d2
