/*
 * slicegcn_native.h -- entry points for hosts that manage memory themselves and for groups of slice models, beside
 * slicegcn.h (same conventions).
 */
#ifndef SLICEGCN_NATIVE_H
#define SLICEGCN_NATIVE_H

#include "slicegcn.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Device memory for the arrays of a graph handle.  alloc returns `bytes` bytes of device memory on the current device,
 * aligned to 256 bytes, or NULL; it is called a handful of times during one build, from the calling thread. */
typedef struct {
    void *ctx;
    void *(*alloc)(void *ctx, size_t bytes);
} slicegcn_allocator;

/* Bytes of scratch memory slicegcn_build_norm_csr_with needs (0 where it returns EINVAL or ERANGE for these sizes and flags). */
size_t slicegcn_build_workspace_bytes(int64_t n_edges, int64_t n_nodes, uint32_t flags);

/* slicegcn_build_norm_csr with the caller's memory.  allocator: where the handle's arrays come from; the caller gives
 * that memory back after slicegcn_graph_destroy, which then frees no device memory (NULL: the library allocates and
 * frees it).  ws: scratch memory, free again when the call returns (NULL: allocated and freed inside).  Device
 * allocations cost as much as the build itself and more, so a host with a caching allocator passes both.
 * EINVAL / ERANGE as slicegcn_build_norm_csr; EWORKSPACE: ws too small; ENOMEM: the allocator returned NULL. */
int slicegcn_build_norm_csr_with(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_nodes, uint32_t flags,
                                 const slicegcn_allocator *allocator, void *ws, size_t ws_bytes, void *stream,
                                 slicegcn_graph **out);

/* ---------------------------------------------------------------------------------------
 * One layer of up to SLICEGCN_MAX_GROUP slice models of equal shape in one set of launches (slicegcn_layer_fwd and
 * slicegcn_layer_bwd for each of them; on a small graph a slice model's kernels fill a fraction of the chip).  A slice's
 * results do not depend on the slices it shares a call with.  In the transform-first order the weight gradients of few rows
 * (n * max(w_in, w_out) <= 2^19) are summed over shorter blocks of rows here than by slicegcn_layer_bwd, whose workspace has no
 * room for more partial sums: they agree up to rounding; everything else is bitwise the same.
 *   enc  : row added to the output outside the activation, beside b_self (the slice encoding), or NULL
 *   denc : receives the column sums of dHout as well (the gradient of enc, equal to db_self), or NULL; both need W_self
 * No slice's output may overlap an operand of another slice of the call.
 * ld*: leading dimensions common to the group (ldgo of dHout, ldgi of dHin).  The forward pass uses Hin, Hout, Z, mask,
 * the backward pass Hin, Z, mask, dHout, dHin (NULL in every entry: not wanted) and grads. */
#define SLICEGCN_MAX_GROUP 8
typedef struct {
    slicegcn_layer_params params;
    const float *enc;
    const float *Hin;
    float *Hout;
    float *Z;
    uint32_t *mask;
    const float *dHout;
    float *dHin;
    slicegcn_layer_grads grads;
    float *denc;
} slicegcn_layer_io;

typedef struct {
    slicegcn_layer_desc desc;
    int32_t count;
    int64_t ldi, ldo, ldz, mask_words, ldgo, ldgi;
} slicegcn_layer_group;

size_t slicegcn_layers_fwd_workspace_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *desc, int32_t count);
size_t slicegcn_layers_bwd_workspace_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *desc, int need_dHin, int32_t count);
int slicegcn_layers_fwd(const slicegcn_graph *g, const slicegcn_layer_group *group, const slicegcn_layer_io *io /* HOST [count] */,
                        void *ws, size_t ws_bytes, void *stream);
int slicegcn_layers_bwd(const slicegcn_graph *g, const slicegcn_layer_group *group, const slicegcn_layer_io *io /* HOST [count] */,
                        void *ws, size_t ws_bytes, void *stream);

/* slicegcn_linear_bwd takes a larger workspace than it requires: with this many bytes its reductions over the nodes are
 * split as finely as they gain from (0 on bad input).  The last bits of dW and db depend on the split, and so on ws_bytes. */
size_t slicegcn_linear_bwd_full_workspace_bytes(int64_t n, int32_t w_in, int32_t w_out);

/* slicegcn_accumulate over 1 to SLICEGCN_MAX_GROUP sources in one sweep: dst[:, 0:w] += srcs[0], then srcs[1], ... (the
 * additions of the single calls in the same order).  srcs: HOST array of DEVICE pointers with leading dimension lds. */
int slicegcn_accumulate_many(float *dst, int64_t ldd, const float *const *srcs, int32_t count, int64_t lds, int64_t n, int32_t w,
                             void *stream);

#ifdef __cplusplus
}
#endif
#endif /* SLICEGCN_NATIVE_H */
