// sw_uf.h -- lock-free union-find on parent arrays in LDS (workgroup scope)
// and in global memory (device scope).  Roots are the smallest index of
// their set: a root is linked under the root with the smaller index, so
// every parent is smaller than its child and the structure stays a forest
// whatever order concurrent unions run in (g_union can link in another order).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swmi {

__device__ __forceinline__ uint32_t lds_load(uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_store(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Root of a once the unions are done (read-only).
__device__ __forceinline__ uint32_t lds_find(uint32_t *par, uint32_t a) {
    while (true) {
        const uint32_t p = lds_load(&par[a]);
        if (p == a) return a;
        a = p;
    }
}
// Both finds advance together, one level per round of loads, with path
// splitting: every entry passed is re-pointed at its grandparent, which is an
// ancestor whatever other unions did meanwhile (a plain store: an entry that
// was not a root never is again).  The two paths meeting below their roots (a
// common parent) already shows one set.
__device__ __forceinline__ void lds_union(uint32_t *par, uint32_t a, uint32_t b) {
    while (true) {
        uint32_t pa = lds_load(&par[a]), pb = lds_load(&par[b]);
        while (pa != a || pb != b) {
            if (pa == pb) return;
            const uint32_t ga = lds_load(&par[pa]), gb = lds_load(&par[pb]);
            if (ga != pa) lds_store(&par[a], ga);
            if (gb != pb) lds_store(&par[b], gb);
            a = pa;
            b = pb;
            pa = ga;
            pb = gb;
        }
        if (a == b) return;
        if (a > b) { const uint32_t tmp = a; a = b; b = tmp; }
        uint32_t expected = b;
        if (__hip_atomic_compare_exchange_strong(&par[b], &expected, a, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
            return;
    }
}

// The tile and brick kernels' parent words hold byte offsets into the LDS array
// (so a parent is directly a load address) and carry other data in their high
// halves (a work list while the unions run).
__device__ __forceinline__ uint32_t *word_at(uint32_t *base, uint32_t off) {
    return reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(base) + off);
}

// Union of the sets of the words at byte offsets a and b: parents are the
// low 16 bits, and the compare-and-swap that links the larger root under the
// smaller keeps the high half it read.  A failed swap (another lane linked
// the root, or the high half changed) resumes from what it found.
__device__ __forceinline__ void lds_union_lo(uint32_t *par, uint32_t a, uint32_t b) {
    while (true) {
        uint32_t wa = lds_load(word_at(par, a)), wb = lds_load(word_at(par, b));
        uint32_t pa = wa & 0xFFFFu, pb = wb & 0xFFFFu;
        while (pa != a || pb != b) {
            a = pa;
            b = pb;
            wa = lds_load(word_at(par, a));
            wb = lds_load(word_at(par, b));
            pa = wa & 0xFFFFu;
            pb = wb & 0xFFFFu;
        }
        if (a == b) return;
        const bool ahi = a > b;
        const uint32_t hi = ahi ? a : b, lo = ahi ? b : a;
        uint32_t expected = ahi ? wa : wb;
        const uint32_t desired = (expected & 0xFFFF0000u) | lo;
        if (__hip_atomic_compare_exchange_strong(word_at(par, hi), &expected, desired, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
            return;
        a = lo;
        b = expected & 0xFFFFu;
    }
}

// Low half (the parent) and high half of the word at byte offset off, each
// read on its own (16-bit loads; the halves are little-endian).
__device__ __forceinline__ uint32_t lo16_at(uint32_t *base, uint32_t off) {
    return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(base) + off);
}
__device__ __forceinline__ uint32_t hi16_at(uint32_t *base, uint32_t off) {
    return *reinterpret_cast<const uint16_t *>(reinterpret_cast<const char *>(base) + off + 2u);
}

// Root (byte offset) of the word at byte offset a once the unions are done.
__device__ __forceinline__ uint32_t lds_root_b(uint32_t *par, uint32_t a) {
    while (true) {
        const uint32_t p = lds_load(word_at(par, a)) & 0xFFFFu;
        if (p == a) return a;
        a = p;
    }
}

__device__ __forceinline__ uint32_t g_load(uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void g_store(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Orders in which g_union links: ByIndex, the smallest index of a set is its
// root; ByBits, the smallest bit-reversed one (for sets whose smallest site is
// gathered separately).
struct ByIndex {
    static __device__ __forceinline__ bool before(uint32_t a, uint32_t b) { return a < b; }
};
struct ByBits {
    static __device__ __forceinline__ bool before(uint32_t a, uint32_t b) { return __brev(a) < __brev(b); }
};
// Union in global memory, as lds_union.
template <class Order = ByIndex>
__device__ __forceinline__ void g_union(uint32_t *par, uint32_t a, uint32_t b) {
    while (true) {
        uint32_t pa = g_load(&par[a]), pb = g_load(&par[b]);
        while (pa != a || pb != b) {
            if (pa == pb) return;
            const uint32_t ga = g_load(&par[pa]), gb = g_load(&par[pb]);
            if (ga != pa) g_store(&par[a], ga);
            if (gb != pb) g_store(&par[b], gb);
            a = pa;
            b = pb;
            pa = ga;
            pb = gb;
        }
        if (a == b) return;
        if (Order::before(b, a)) { const uint32_t tmp = a; a = b; b = tmp; }
        uint32_t expected = b;
        if (__hip_atomic_compare_exchange_strong(&par[b], &expected, a, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return;
    }
}

}  // namespace swmi
