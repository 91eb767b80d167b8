// sc_union.hpp -- union-find walks over 32-bit parents that several threads read and relink at once.
//
// M gives the accesses, each atomic by itself: load(i), store(i, v), min(i, v) -> the value before.
// A parent is never larger than its entry, a root is its own parent, and a relinked entry keeps an
// ancestor, so every walk ends at the root that its entry has, or had while unions went on.
#pragma once

#include <cstdint>

namespace sc {

// Root of x, halving the path: an entry on the way is relinked to its grandparent.  The store may
// come late: an entry that another thread has pointed at its root meanwhile can be left with an
// inner node of the tree.  So while such walks run, take roots from what they return, never from
// the entries.
template <typename M>
__device__ __forceinline__ uint32_t union_root_halving(M m, uint32_t x)
{
    while (true) {
        const uint32_t p = m.load(x);
        if (p == x) return x;
        const uint32_t g = m.load(p);
        if (g == p) return p;
        m.store(x, g);
        x = g;
    }
}

// Joins the sets of a and b.  Both ends are followed together, so that their loads are in flight at
// once, and both paths are halved: where many links join one large set, the roots of its parts form
// long chains.
template <typename M>
__device__ __forceinline__ void union_unite(M m, uint32_t a, uint32_t b)
{
    while (true) {
        while (true) {
            if (a == b) return;
            const uint32_t pa = m.load(a), pb = m.load(b);
            if (pa == a && pb == b) break;
            const uint32_t ga = m.load(pa), gb = m.load(pb);
            if (pa != a && ga != pa) m.store(a, ga);
            if (pb != b && gb != pb) m.store(b, gb);
            a = ga;
            b = gb;
        }
        if (a > b) { const uint32_t t = a; a = b; b = t; }
        const uint32_t old = m.min(b, a);
        if (old == b) return;
        b = old;
    }
}

// Points x at its root, once the unions are done.  The walk only reads, so x is written here alone,
// and if every entry is settled by one thread, all of them hold their roots afterwards.
template <typename M>
__device__ __forceinline__ void union_settle(M m, uint32_t x)
{
    uint32_t r = x;
    for (uint32_t p = m.load(r); p != r; p = m.load(r)) r = p;
    m.store(x, r);
}

}  // namespace sc
