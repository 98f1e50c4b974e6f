/*
 * swan_layer.h -- what the layer code (layer.py) calls beyond swan.h, in the
 * same library and under the conventions stated there.
 */
#ifndef SWAN_LAYER_H
#define SWAN_LAYER_H

#include "swan.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * `count` problems of swan_calibrate_rotation at once, side by side on the GPU
 * (the rotations of a layer's heads; the solver of one occupies one compute
 * unit): rows holds the problems' rows one after another, n_rows_host[count] of
 * each (>= 1); P_out [count][d][d], sigma_out [count][d] or NULL, workspace
 * count times what swan_calibrate_workspace_bytes says.  Every problem's result
 * is the same as from a call of its own.
 */
swan_status swan_calibrate_rotations(const float* rows, int32_t count,
                                     const int64_t* n_rows_host, int32_t d, float* P_out,
                                     float* sigma_out, void* workspace, size_t workspace_bytes,
                                     void* stream);

#ifdef __cplusplus
}
#endif

#endif /* SWAN_LAYER_H */
