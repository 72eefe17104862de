/*
 * slicegcn_native.h -- entry points for hosts that manage memory themselves, beside slicegcn.h (same conventions).
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

/* Bytes of scratch memory slicegcn_build_norm_csr_with needs (0 on bad input). */
size_t slicegcn_build_workspace_bytes(int64_t n_edges, int64_t n_nodes, uint32_t flags);

/* slicegcn_build_norm_csr with the caller's memory.  allocator: where the handle's arrays come from; the caller gives
 * that memory back after slicegcn_graph_destroy, which then frees no device memory (NULL: the library allocates and
 * frees it).  ws: scratch memory, free again when the call returns (NULL: allocated and freed inside).  Device
 * allocations cost more than the build itself on most graphs, so a host with a caching allocator passes both.
 * EINVAL / ERANGE as slicegcn_build_norm_csr; EWORKSPACE: ws too small; ENOMEM: the allocator returned NULL. */
int slicegcn_build_norm_csr_with(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_nodes, uint32_t flags,
                                 const slicegcn_allocator *allocator, void *ws, size_t ws_bytes, void *stream,
                                 slicegcn_graph **out);

#ifdef __cplusplus
}
#endif
#endif /* SLICEGCN_NATIVE_H */
