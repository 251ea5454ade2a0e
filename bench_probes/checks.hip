// Checks of the step's per-element code (csrc/elem.h, csrc/exact.h) on the
// device, declared in madd_probes.h.  They call the functions the step kernels
// are built from, not copies of them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "elem.h"
#include "madd_probes.h"

namespace {

using namespace madd_detail;

template <int WF>
constexpr bool fp4() {
  return WF == WF_MXFP4 || WF == WF_NVFP4;
}

// One quad per thread: the step's four elements as the kernels take them, the
// general arithmetic on its own, and which of the two the quad took.
template <bool CLAMP>
__global__ __launch_bounds__(256) void step_path_kernel(
    const float* __restrict__ w, const float* __restrict__ g, const float* __restrict__ m,
    const float* __restrict__ v, const float* __restrict__ ve, int64_t quads,
    const Scalars* __restrict__ sp, float* __restrict__ got, float* __restrict__ general,
    uint8_t* __restrict__ took) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= quads) return;
  const Scalars s = *sp;
  float w4[4], wn[4];
  f4 g4, m4, v4, ve4;
  for (int k = 0; k < 4; ++k) {
    w4[k] = w[4 * q + k];
    g4[k] = g[4 * q + k];
    m4[k] = m[4 * q + k];
    v4[k] = v[4 * q + k];
    ve4[k] = ve[4 * q + k];
  }
  took[q] = step_four<CLAMP, false, false>(w4, g4, m4, v4, ve4, wn, s) ? 1 : 0;
  for (int k = 0; k < 4; ++k) {
    float mk = m[4 * q + k], vk = v[4 * q + k], vek = ve[4 * q + k], ge;
    moments_elem(w4[k], g4[k], mk, vk, vek, ge, s);
    got[4 * q + k] = wn[k];
    general[4 * q + k] = weight_elem<CLAMP>(w4[k], ge, add_update(mk, vk, s), vek, s);
  }
}

// A minifloat code from the value grid: |x| scaled so that the spacing of its
// binade is 1, rounded to an integer.  `f16`: the top 16 bits of the fraction
// that the stochastic rule compares.
template <int M, int BIAS, int EMIN>
struct Grid {
  uint32_t base, sign, f16, k, rne;
  __device__ __forceinline__ Grid(float x, float top, int signbit) {
    const float a = fminf(fabsf(x), top);
    const int e = (int)(__float_as_uint(a) >> 23) - 127, se = (e > EMIN ? e : EMIN) - M;
    const float q = ldexpf(a, -se), fl = floorf(q);
    base = (uint32_t)(se + M + BIAS - 1) << M;
    sign = (__float_as_uint(x) >> 31) << signbit;
    k = (uint32_t)fl;
    f16 = (uint32_t)((q - fl) * 65536.0f);
    rne = sign | (base + (uint32_t)rintf(q));
  }
  // the draws on both sides of the threshold (both below it when f16 is 0)
  __device__ __forceinline__ uint32_t draw(int side) const {
    return f16 ? 65536u - f16 - (uint32_t)side : (side ? 0u : 65535u);
  }
  __device__ __forceinline__ uint32_t sr(int side) const {
    return sign | (base + k + (f16 + draw(side) >= 65536u ? 1u : 0u));
  }
};

// The step's four-element encoders on every fp32 but NaN, in every position of
// the group: element k of a group takes bits 30-31 of its pattern from k and
// the rotation.  c: see madd_check_encoders.
template <int WF, int M, int BIAS, int EMIN>
__device__ __forceinline__ void check_mini(const float (&x)[4], float top, unsigned long long& rne,
                                           unsigned long long& sr) {
  constexpr int kBits = fp4<WF>() ? 4 : 8;
  typedef Grid<M, BIAS, EMIN> G;
  const G g[4] = {G(x[0], top, kBits - 1), G(x[1], top, kBits - 1), G(x[2], top, kBits - 1),
                  G(x[3], top, kBits - 1)};
#pragma unroll
  for (int rot = 0; rot < 4; ++rot) {
    float y[4];
    uint32_t r[4], want = 0u, got;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      y[k] = x[(k + rot) & 3];
      r[k] = 0u;
      want |= g[(k + rot) & 3].rne << (kBits * k);
    }
    if constexpr (fp4<WF>()) got = enc_e2m1x4<false>(y, r);
    else got = enc_fp8x4<WF, false>(y, r);
    rne += got != want;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      want = 0u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        r[k] = g[(k + rot) & 3].draw(side);
        want |= g[(k + rot) & 3].sr(side) << (kBits * k);
      }
      if constexpr (fp4<WF>()) got = enc_e2m1x4<true>(y, r);
      else got = enc_fp8x4<WF, true>(y, r);
      sr += got != want;
    }
  }
}

// 2^24 threads, 64 groups each.
__global__ __launch_bounds__(256) void encoders_kernel(unsigned long long* c) {
  const uint32_t tid = blockIdx.x * 256u + threadIdx.x;
  unsigned long long n[8] = {};
  for (uint32_t j = 0; j < 64u; ++j) {
    uint32_t u[4];
    float x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      u[k] = (tid * 64u + j) | ((uint32_t)k << 30);
      x[k] = __uint_as_float(u[k]);
      if (x[k] != x[k]) x[k] = __uint_as_float((u[k] & 0x80000000u) | 0x3F800000u);
    }
    check_mini<WF_E4M3, 3, 7, -6>(x, 448.0f, n[0], n[1]);
    check_mini<WF_E5M2, 2, 15, -14>(x, 57344.0f, n[2], n[3]);
    check_mini<WF_MXFP4, 1, 1, 0>(x, 6.0f, n[4], n[5]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // bf16 pairs; a NaN is the canonical one
      const uint32_t a = (u[k] & 0x7FFFFFFFu) > 0x7F800000u ? 0x7FC00000u : u[k];
      const uint32_t b = (u[(k + 1) & 3] & 0x7FFFFFFFu) > 0x7F800000u ? 0x7FC00000u : u[(k + 1) & 3];
      const uint32_t want = ((a + 0x7FFFu + ((a >> 16) & 1u)) >> 16) |
                            ((b + 0x7FFFu + ((b >> 16) & 1u)) & 0xFFFF0000u);
      n[6] += enc_bf16x2(__uint_as_float(a), __uint_as_float(b), false, 0u, 0u) != want;
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const uint32_t la = a & 0xFFFFu, lb = b & 0xFFFFu;
        const uint32_t ra = la ? 65536u - la - side : (side ? 0u : 65535u),
                       rb = lb ? 65536u - lb - side : (side ? 0u : 65535u);
        n[7] += enc_bf16x2(__uint_as_float(a), __uint_as_float(b), true, ra, rb) !=
                (((a + ra) >> 16) | ((b + rb) & 0xFFFF0000u));
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (n[k]) atomicAdd(&c[k], n[k]);
  if (threadIdx.x == 0) atomicAdd(&c[8], 256ull * 64ull);  // this workgroup's groups
}

}  // namespace

extern "C" int32_t madd_check_encoders(uint64_t* counters, void* stream) {
  if (!counters) return -1;
  hipLaunchKernelGGL(encoders_kernel, dim3(65536), dim3(256), 0, (hipStream_t)stream,
                     (unsigned long long*)counters);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

extern "C" int32_t madd_probe_step_path(const float* w, const float* g, const float* m,
                                        const float* v, const float* ve, int64_t quads,
                                        const void* scalars, int32_t clamp, float* got,
                                        float* general, uint8_t* took, void* stream) {
  if (quads < 0 || quads > ((int64_t)1 << 30) || (clamp != 0 && clamp != 1)) return -1;
  if (quads == 0) return 0;
  if (!w || !g || !m || !v || !ve || !scalars || !got || !general || !took) return -1;
  const dim3 grid((unsigned)((quads + 255) / 256)), block(256);
  const Scalars* sp = (const Scalars*)scalars;
  if (clamp)
    hipLaunchKernelGGL(step_path_kernel<true>, grid, block, 0, (hipStream_t)stream, w, g, m, v, ve,
                       quads, sp, got, general, took);
  else
    hipLaunchKernelGGL(step_path_kernel<false>, grid, block, 0, (hipStream_t)stream, w, g, m, v, ve,
                       quads, sp, got, general, took);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}
