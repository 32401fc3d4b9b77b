/*
 * qfc_experimental - knobs and a probe of libqfc.so that are NOT part of its interface.
 *
 * qfc_tune is used by this repository's tests and parameter sweeps to force a
 * kernel variant that the dispatcher would not pick for a given shape (so that
 * every variant can be checked on small inputs); qfc_probe_mfma is a
 * measurement aid of bench.py.  Nothing here follows a passage of the paper,
 * nothing here is needed to use the library, and it may change without
 * notice.  Production callers include qfc.h only.
 */
#ifndef QFC_EXPERIMENTAL_H
#define QFC_EXPERIMENTAL_H

#include <stdint.h>

#include "qfc.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Set one process-wide tunable (each is a single atomic integer; a call that is
 * being enqueued on another thread sees either the old or the new value of each
 * key, never a torn one).  Unknown keys are ignored.
 *   key 0  target number of wavefronts of a decode launch (0 = automatic: 8192 up to two token rows, 2048 above)
 *   key 1  most row tiles a decode workgroup walks (0 = automatic: 2 up to two token rows, 4 above)
 *   key 2  prefill kernel by number (0 = automatic).  Binary16 activations: 9 the kernel for any K, 31 .. 37 the forms of the main
 *          kernel: 32, 64, 96, 128 token rows per workgroup, and, for K of 256 and more, 128, 64 and 96 with K in two halves.  int8
 *          activations: int8 weights 4 both operands staged, 10 and 12 weights straight into registers with 128 and 64 token rows and 256
 *          channels per workgroup, 13 and 14 the same with 128 channels and K in two parts; int4 weights 20, 21 and 23 as 4, 10 and 12, 24
 *          and 25 128 channels and 64 token rows with K in two and four parts.  Any number but 0 leaves out the kernels for few token
 *          rows; one that names no kernel of the call's formats and size leaves the choice among the others
 *   key 3  token rows per workgroup of the activation quantization kernel (0 = automatic; 2, 4, 8)
 *   key 4  half-unit items of the decode kernel (-1 automatic, 0 never, 1 where possible)
 *   key 5  (without effect)
 *   key 6  causal walks of prefill attention cut into chunks (-1 automatic, 0 never, 1 always, 2, 3, 4, 6, 8 into so many);
 *          qfc_attention_workspace_size follows the value set when it is called
 *   key 7  products of few token rows (from 9): most wavefronts per workgroup (0 = automatic)
 *   key 8  the same: row tiles per workgroup (0 = automatic; 1 .. 8)
 *   key 9  the same: largest number of token rows they are used for (-1 automatic, 0 never)
 *   key 10 gated output at M <= 8: pairs of row tiles per decode workgroup (0 = automatic; 1, 2)
 *   key 11 as key 7: blocks the token rows are cut into at least (0 = automatic)
 *   key 12 attention with at most 16 query rows per KV head: workgroups per KV head (0 = automatic; 1 .. 64)
 *   key 13 attention with more than 16 query rows per KV head: blocks of 16 (-1 automatic, 0 never, 1 always)
 *   key 14 prefill attention: wavefronts that share the walk of the same query rows (0 = automatic; 1, 2) */
void qfc_tune(int32_t key, int32_t value);

/* Measurement probe (bench.py --probe-mfma): `workgroups` workgroups of four wavefronts each issue
 * 32 * iters back-to-back MFMAs from registers, no memory traffic (kind 0: v_mfma_i32_32x32x32_i8,
 * 65536 operations each; 1: v_mfma_f32_32x32x16_f16, 32768; 4: v_mfma_i32_16x16x64_i8, 32768; 5:
 * v_mfma_f32_16x16x32_f16, 16384), with constant operands (random_operands = 0), operands of random
 * bits used in rotation (1), codes of normal values (int8) or normal values (binary16) (2), or the
 * same with int4 codes as the first operand (3).  ticks (device, 8-byte
 * aligned, 2 * workgroups entries, written by the kernel): per workgroup the shader-clock ticks
 * and the ticks of the constant 100 MHz counter over the loop.  The caller times the launch.
 * Errors: QFC_ERR_INVALID_ARG (kind, iters outside 1 .. 2^22, workgroups outside 1 .. 4096, null),
 * QFC_ERR_ALIGNMENT, QFC_ERR_HIP. */
qfc_status_t qfc_probe_mfma(int32_t kind, int32_t random_operands, int32_t iters, int32_t workgroups,
                            uint64_t *ticks, void *stream);

#ifdef __cplusplus
}
#endif
#endif /* QFC_EXPERIMENTAL_H */
