// Union-find labels of bodies: lab[b] < 0 for a body in no pair, b for a root, else a smaller body
// of the same component.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace genga {

// lab[] is read with device-coherent atomic loads, so what other waves' atomics wrote (performed in
// L2) is seen without cache maintenance.
__device__ __forceinline__ int uf_load(int32_t *lab, int a)
{
    return __hip_atomic_load(&lab[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int uf_root(int32_t *lab, int a)
{
    int r = uf_load(lab, a);
    while (r != a) {
        a = r;
        r = uf_load(lab, a);
    }
    return r;
}

// Root of a with path halving: every visited node is pointed at its grandparent.  Labels only ever
// move to a smaller index of the same tree (roots are linked under smaller roots, by
// compare-and-swap), and only nodes that are no longer roots are pointed elsewhere, so a halving
// step that races with a link or another halving still leaves a valid ancestor.
__device__ __forceinline__ int uf_find(int32_t *lab, int a)
{
    int p = uf_load(lab, a);
    while (p != a) {
        const int gp = uf_load(lab, p);
        if (gp != p) __hip_atomic_store(&lab[a], gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a = gp;
        p = uf_load(lab, a);
    }
    return a;
}

} // namespace genga
