// Checks of the step's per-element code (csrc/elem.h, csrc/exact.h) on the
// device, declared in madd_probes.h.  They call the functions the step kernels
// are built from, not copies of them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "elem.h"
#include "madd_probes.h"

namespace {

using namespace madd_detail;

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

}  // namespace

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
