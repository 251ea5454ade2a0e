/*
 * madd_probes.h -- C ABI of libmadd_probes.so: device probes for AMD
 * Instinct MI355X (gfx950) that the benchmark and the tests use.  Not part
 * of the optimizer.
 *
 * madd_ceiling_stream: the empirical bandwidth ceiling of the M+Adam step.
 * The step (include/madd.h) is bound by HBM bandwidth: per element it
 * streams the weight code, the gradient and the three moments in and the
 * weight code and the three moments out (for bf16 weights and fp32 moments
 * 18 bytes read and 14 written).  The probe moves exactly those bytes with
 * the step kernel's work mapping (2048 elements per 256-thread workgroup,
 * four consecutive elements per thread and 1024-element sub-tile,
 * non-temporal 8/16-byte accesses) and no arithmetic.  Every buffer is
 * written back unchanged (each value is XORed with the gradient's bits
 * masked by a runtime zero), so the probe can run on live optimizer state.
 *
 * madd_stream_modes: plain streams in the same access shape (a 256-thread
 * workgroup per 8 KiB tile, 16 bytes per thread in each 4 KiB half,
 * non-temporal): read only, write only, or copy.  Together with the
 * ceiling probe they place the step between what HBM delivers for reads
 * alone, for writes alone and for the step's own read:write mix.
 *
 * madd_probe_bf16_rounding: the step kernel rounds fp32 to bf16 with the
 * v_cvt_pk_bf16_f32 (round to nearest-even) and v_cvt_sr_bf16_f32
 * (stochastic) instructions.  The probe runs both on all 2^32 fp32 bit
 * patterns and counts disagreements with the integer definitions of the
 * two roundings: RNE(u) = (u + 0x7FFF + ((u >> 16) & 1)) >> 16 and
 * SR(u, r16) = (u + r16) >> 16 with the draw r16 in the high half of the
 * instruction's random operand, and checks that the canonical quiet NaN
 * 0x7FC00000 converts to 0x7FC0 under both.
 */
#ifndef MADD_PROBES_H
#define MADD_PROBES_H

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* One pass over n elements: read w (bf16 codes), g (fp32), m, v, ve
 * (state_bytes = 4: fp32, 2: bf16 codes), write w, m, v, ve.
 * All pointers are DEVICE pointers, 16-byte aligned, owned by the caller;
 * n >= 0.  Enqueued on `stream` (hipStream_t as void*).
 * Returns 0 on success, -1 for an invalid argument (NULL pointer, n < 0,
 * state_bytes not 2 or 4), -2 for an unaligned pointer, -4 when the launch
 * fails; nothing is launched on an error. */
int32_t madd_ceiling_stream(void* w, const float* g, void* m, void* v, void* ve,
                            int32_t state_bytes, int64_t n, void* stream);

/* One pass of a plain stream over `bytes` bytes (a positive multiple of
 * 8192): mode 0 reads a (and writes at most the first 4 KiB of b, and only
 * when an XOR of what it read equals a fixed key, which keeps the loads
 * alive), mode 1 writes b, mode 2 copies a to b.  DEVICE pointers, 16-byte
 * aligned, owned by the caller; a may be NULL in mode 1.  Enqueued on
 * `stream`.  Returns 0, -1 for an invalid argument (unknown mode, bad size,
 * NULL pointer), -2 for an unaligned pointer, -4 when the launch fails;
 * nothing is launched on an error. */
int32_t madd_stream_modes(int32_t mode, const void* a, void* b, int64_t bytes, void* stream);

/* Exhaustive check of the two bf16 conversion instructions.
 * counters: DEVICE array of 4 uint64 values owned by the caller, which the
 * caller zeroes before the call; on completion they hold
 *   [0] non-NaN inputs where v_cvt_pk_bf16_f32 differs from RNE(u),
 *   [1] non-NaN inputs where v_cvt_sr_bf16_f32 differs from SR(u, r16)
 *       (r16: a fixed hash of u, so every input meets a different draw),
 *   [2] conversions of 0x7FC00000 (both instructions, with every draw of a
 *       sample of 2^16 draws) that do not give 0x7FC0,
 *   [3] the number of inputs examined (2^32).
 * Enqueued on `stream`.  Returns 0, -1 for a NULL pointer, -4 when the
 * launch fails. */
int32_t madd_probe_bf16_rounding(uint64_t* counters, void* stream);

/* The range-limited square root and division of csrc/exact.h against the
 * general operations.
 * counters: DEVICE array of 4 uint64 values owned by the caller, which the
 * caller zeroes before the call; on completion they hold
 *   [0] inputs +-0 and finite x >= 2^-46 where the square root differs,
 *   [1] inputs 2^-126 <= |x| < 2^126 where the refined reciprocal is not 1 / x,
 *   [2] pairs of significands where the quotient differs (every denominator,
 *       1024 numerators each: 512 hashed, 512 around it), and quotients of
 *       -0 that are not -0,
 *   [3] the number of bit patterns examined for [0] and [1] (2^32).
 * Enqueued on `stream`.  Returns 0, -1 for a NULL pointer, -4 when the
 * launch fails. */
int32_t madd_check_exact_ops(uint64_t* counters, void* stream);

/* The quotient of csrc/exact.h against the general division: every numerator
 * significand over the `count` (at most 65536) denominator significands from
 * `first` on, of 2^23.  counters: DEVICE array of 2 uint64 values owned by the
 * caller, added to: [0] pairs that differ, [1] pairs examined.  Enqueued on
 * `stream`.  Returns 0, -1 for an invalid argument, -4 when the launch fails. */
int32_t madd_check_quotients(int32_t first, int32_t count, uint64_t* counters, void* stream);

/* The step's arithmetic (csrc/elem.h) on `quads` groups of four elements, and
 * which of its two forms each group took.
 * w, g, m, v, ve: DEVICE fp32 arrays of 4 quads elements (weight values, the
 * gradients, the moments before the step); scalars: DEVICE copy of
 * madd_prepare_scalars' bytes; clamp: 1 applies g_max and w_max.
 * got: the new weights as the kernels compute them; general: the same from the
 * general square root and division; took: one byte per group, 1 if it fell
 * back to those.  All owned by the caller.  Enqueued on `stream`.  Returns 0,
 * -1 for an invalid argument, -4 when the launch fails. */
int32_t madd_probe_step_path(const float* w, const float* g, const float* m, const float* v,
                             const float* ve, int64_t quads, const void* scalars, int32_t clamp,
                             float* got, float* general, uint8_t* took, void* stream);

/* The encoders the step's stores are made with (csrc/elem.h: enc_fp8x4,
 * enc_e2m1x4, enc_bf16x2) against the value grids and the integer rules, on
 * every fp32 but NaN in every position of a group, stochastically with the
 * draws on both sides of each element's threshold; for bf16 also the canonical
 * NaN.
 * counters: DEVICE array of 9 uint64 values owned by the caller, which the
 * caller zeroes before the call; on completion they hold the groups that
 * differ: [0] E4M3 to nearest, [1] E4M3 stochastic, [2], [3] E5M2, [4], [5]
 * E2M1, [6], [7] bf16 pairs, and [8] the number of groups of four patterns
 * (2^30, each in four rotations).  Enqueued on `stream`.  Returns 0, -1 for a
 * NULL pointer, -4 when the launch fails. */
int32_t madd_check_encoders(uint64_t* counters, void* stream);

/* madd_probe_delay: one wave on `stream` that sleeps `sleeps` times (each
 * s_sleep 127, about 8k cycles, ~3.5 us) and exits.  The benchmark enqueues
 * it ahead of a run of short steps so that the host has queued them all
 * before the first starts, and the events between steps time the GPU alone.
 * Returns -1 for sleeps outside [0, 2^20], -3 if the launch fails. */
int32_t madd_probe_delay(int32_t sleeps, void* stream);

#ifdef __cplusplus
}
#endif

#endif /* MADD_PROBES_H */
