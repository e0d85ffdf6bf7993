/*
 * bf_test.h -- test hooks of libbf.  Not for production use: they exist so
 * that the test suite can check host-visible pieces of the kernels and reach
 * code paths that production sizes reach only with very large inputs.  They
 * follow the conventions of bf.h (status returns, bf_last_error).
 */
#ifndef BF_TEST_H
#define BF_TEST_H

#include <stdint.h>

#include "bf.h"

#ifdef __cplusplus
extern "C" {
#endif

/* The Hann window of Eq. 3, W(u) = cos^2(pi u) for u < 1/2, as the gather
 * kernels evaluate it: the library's degree-6 polynomial in w = u^2 (the
 * same host/device function, evaluated on the host in FP32). */
double bf_test_hann_poly(double u2);

/* Cap on the frames one launch of bf_das_adjoint_frames takes (each gradient
 * of a stack goes in launches of at most `cap` frames; 0 = no cap, the
 * default: as many as the plan's partial-sum buffer holds).  Results do not
 * depend on it.  BF_ERR_SHAPE for cap < 0. */
int bf_test_set_stack_cap(bf_plan plan, int32_t cap);

/* Restrict the mirror axes of a plan (bit 0: y, bit 1: x; before its first
 * batched launch) and return the axes its frames then use, so that tests can
 * compare mirrored launches with plain ones. */
int bf_test_set_mirrors(bf_plan plan, int32_t allowed);
/* The mirror axes the frames of a plan use. */
int bf_test_mirror_axes(bf_plan plan);

/* Run a demodulator's calls on the vector units (unit 1), on the matrix cores (2,
 * where its filter fits them) or where the library's rule puts them (0); returns
 * the unit they then run on, 1 or 2. */
int bf_test_demod_unit(bf_demod d, int32_t unit);

/* The launch bf_das would make for a description, on the host alone (no device
 * is needed), with the mirror axes restricted to `allowed`: lds = 0 is the
 * gather kernel; nb counts the traces per batch and mirror copy, mirrors the
 * axes used, blocks the workgroup boxes along x, y and z, refs the delay
 * references of a box. */
typedef struct {
    int32_t lds, mirrors, nb, zp, tile[3], block[3], blocks[3], lmax, groups, adj_groups, refs;
} bf_test_launch;
int bf_test_das_launch(const bf_params *params, int32_t allowed, bf_test_launch *out);

#ifdef __cplusplus
}
#endif
#endif /* BF_TEST_H */
