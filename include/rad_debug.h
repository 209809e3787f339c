/*
 * rad_debug.h - diagnostic entry points of the radiation library (not needed to compute
 * spectra).  Same conventions as rad.h.
 */
#ifndef RAD_DEBUG_H
#define RAD_DEBUG_H

#include "rad.h"

#ifdef __cplusplus
extern "C" {
#endif

/* For each of n revolutions r = in_dev[i] (DEVICE, floats), write to out_dev[4i..4i+3]
 * (DEVICE) the sine and cosine of 2*pi*r from the hardware transcendental unit used to
 * seed the frequency walk, then from the library sincospi used for the per-particle
 * rotation factor.  Lets a test measure both against FP64 references.  Stream-ordered. */
int rad_debug_trig_probe(const float* in_dev, float* out_dev, int n, void* stream);

/* One accumulate launch of a push. */
typedef struct rad_debug_launch {
    int32_t kernel;        /* 0: fixed tiles, 1: lanes laid out at run time, 2: matrix cores */
    int32_t k0, n_omega;   /* the frequencies that it sums                                  */
    rad_tile tile;         /* its launch shape (kernel 2 has none)                          */
    int32_t splits;        /* particle splits, each with a partial sum of its own           */
    int64_t per_split;     /* particles of a split                                          */
    int32_t chunk;         /* particles staged at a time                                    */
    int32_t weights_at;    /* kernel 1: where the table of weights starts in LDS [B]        */
    int32_t lds_bytes;     /* kernels 0 and 1: LDS of a workgroup                           */
} rad_debug_launch;

/* The accumulate launches that a push of n_particles (all steps together) makes into a grid
 * of this description on a device of `cus` compute units, with `tile` set or (NULL) none:
 * the first max_launches of them to out, their number to *n_launches.  Host only: needs no
 * device. */
int rad_debug_plan(const rad_grid_desc* d, const rad_tile* tile, int32_t cus, int64_t n_particles,
                   rad_debug_launch* out, int32_t max_launches, int32_t* n_launches);

#ifdef __cplusplus
}
#endif

#endif /* RAD_DEBUG_H */
