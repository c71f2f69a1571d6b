/* What the library would launch, for programs that measure it (bench.py, tests). Not part of the operator ABI of
 * purine.h: an answer may change with any version of the library. Host code only. */
#ifndef PURINE_INTROSPECT_H
#define PURINE_INTROSPECT_H
#include "purine.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Matrix-core products that a pass (PURINE_CONV_*) executes per multiplication of its layer: 1 where it multiplies in
 * the layer's own type, 6 where an F32 pass multiplies bf16 parts (whichever kernel it runs on). 0 for an illegal shape. The launch's own plan for
 * dense tensors. */
int purine_conv_matrix_products(int pass, const purine_conv_desc* desc, const int64_t x_dim[4],
                                const int64_t w_dim[4], int32_t dtype);

/* Which of the kernels that the test hooks (-11) to (-13) of purine_debug_force_tile name a pass runs, or 0 for any other (and for
 * an illegal shape). The launch's own plan for dense tensors, hooks included. */
enum { PURINE_ROUTE_OTHER = 0, PURINE_ROUTE_SMALL_LAUNCH = 1, PURINE_ROUTE_INSIDE_LDS = 2 };
int purine_conv_route(int pass, const purine_conv_desc* desc, const int64_t x_dim[4], const int64_t w_dim[4], int32_t dtype);
int purine_fc_route(int pass, int64_t N, int64_t C, int64_t K, int32_t dtype);

#ifdef __cplusplus
}
#endif
#endif
