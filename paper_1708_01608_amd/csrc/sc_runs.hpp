// sc_runs.hpp -- gas masks as 64-bit words and the runs of their bits: what the labelling
// (sc_label.hip) and the test pass (sc_test.hip) share, with the wave-level sums by key.
#pragma once

#include "sc_device.hpp"
#include "sc_internal.hpp"
#include "sc_union.hpp"

namespace sc {

constexpr int kSeg = 64;

__host__ __device__ __forceinline__ int segs_of(int nx) { return (nx + kSeg - 1) / kSeg; }

// ---- bits of a word --------------------------------------------------------------------------
__device__ __forceinline__ uint64_t below(int p) { return p ? ~0ull >> (64 - p) : 0ull; }

// First bit of the run of `w` that contains bit p.
__device__ __forceinline__ int run_start(uint64_t w, int p)
{
    const uint64_t gap = ~w & below(p);
    return gap ? 64 - __clzll((long long)gap) : 0;
}

// The run of `w` that starts at bit s, as a mask.
__device__ __forceinline__ uint64_t run_at(uint64_t w, int s)
{
    const uint64_t t = ~(w >> s);
    const int len = t ? __ffsll((long long)t) - 1 : 64;
    return below(min(len, 64 - s)) << s;
}

// The scratch of a labelling: the words (one a segment, rows one after the other), then the parents.
// A parent is kept as its entry times two plus the parity of its column, which names the node.
struct LabelScratch {
    uint64_t* words;
    uint32_t* parent;
    uint32_t half;  // parents a row
};
__host__ __device__ __forceinline__ LabelScratch scratch_of(uint32_t* p, const FieldArgs& a)
{
    const size_t words = (size_t)segs_of(a.nx) * a.ny * a.nz;
    return LabelScratch{reinterpret_cast<uint64_t*>(p), p + 2 * words, (uint32_t)(a.nx + 1) / 2};
}
// Code of the run start at column x of row r, and the node of a code.
__device__ __forceinline__ uint32_t code_of(uint32_t r, int x, uint32_t half)
{
    return 2 * (r * half + ((uint32_t)x >> 1)) + ((uint32_t)x & 1);
}
__device__ __forceinline__ uint32_t node_of_code(uint32_t c, uint32_t half, int nx)
{
    const uint32_t e = c >> 1, r = e / half;
    return r * (uint32_t)nx + 2 * (e - r * half) + (c & 1);
}

// Segment `w` of the box: first node, width, row.
struct Seg {
    int64_t n;
    uint32_t r;
    int width, x0, y, z;
};
__device__ __forceinline__ Seg seg_of(int64_t w, const FieldArgs& a)
{
    const uint32_t segs = (uint32_t)segs_of(a.nx), r = (uint32_t)w / segs, s = (uint32_t)w - r * segs;
    Seg g;
    g.x0 = (int)s * kSeg;
    g.width = min(kSeg, a.nx - g.x0);
    g.r = r;
    g.n = (int64_t)r * a.nx + g.x0;
    g.z = (int)(r / (uint32_t)a.ny);
    g.y = (int)(r - (uint32_t)g.z * (uint32_t)a.ny);
    return g;
}

// ---- union-find in LDS -----------------------------------------------------------------------
struct LdsParents {
    uint32_t* p;
    __device__ __forceinline__ uint32_t load(uint32_t i) const
    {
        return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void store(uint32_t i, uint32_t v) const
    {
        __hip_atomic_store(p + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ uint32_t min(uint32_t i, uint32_t v) const
    {
        return atomicMin(p + i, v);
    }
};

// The run starts of a word that fall to one of PARTS lanes: a word of a bubble has one run or two, one
// of a fine mask up to 32, which a single lane would unite one after the other.
template <int PARTS>
__device__ __forceinline__ uint64_t run_starts(uint64_t w, int part)
{
    return w & ~(w << 1) & (~0ull >> (64 - kSeg / PARTS) << kSeg / PARTS * part);
}

// Calls link(sa, sb) once for every pair of touching runs of two adjacent rows: sa, sb the first
// bits of the runs of words A and B, sa among `starts`; `wide` rows touch diagonally too.
template <typename F>
__device__ __forceinline__ void touching_runs(uint64_t A, uint64_t B, uint64_t starts, bool wide,
                                              F link)
{
    const uint64_t reach = wide ? (A | A << 1 | A >> 1) : A;
    if (!(reach & B)) return;
    for (; starts; starts &= starts - 1) {
        const int sa = __ffsll((long long)starts) - 1;
        const uint64_t run = run_at(A, sa);
        uint64_t hit = B & (wide ? (run | run << 1 | run >> 1) : run);
        while (hit) {
            const int sb = run_start(B, __ffsll((long long)hit) - 1);
            hit &= ~run_at(B, sb);
            link(sa, sb);
        }
    }
}

// The rows after a row that its nodes link to (half of the lattice's directions, the other half
// seen from there), and whether along x by one node as well as straight.
template <int Q>
struct RowLinks;
template <>
struct RowLinks<9> {
    static constexpr int n = 1;
    static constexpr int dy[1] = {1}, dz[1] = {0};
    static constexpr bool wide[1] = {true};
};
template <>
struct RowLinks<19> {
    static constexpr int n = 4;
    static constexpr int dy[4] = {1, 0, 1, 1}, dz[4] = {0, 1, 1, -1};
    static constexpr bool wide[4] = {true, true, false, false};
};

// ---- wave-level aggregation of per-node atomics ------------------------------------------------
// Per-node contributions to per-bubble counters arrive from many nodes of the same bubble at
// once; one atomic per node onto a few hundred addresses serialises.  The lanes of a wave that
// carry the same key (a bubble slot, >= 0) sum their values with a butterfly and one lane adds the
// sum: one atomic per key and wave.  Integer sums, so the result does not depend on the
// grouping.  Every lane of the wave must call these (the loops below are wave-uniform).
__device__ __forceinline__ long long wave_sum_i64(long long v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Where a wave meets many bubbles, one after the other is a long serial chain (a butterfly of four
// sums some 0.5 us), and few of its atomics meet on one address anyway: keys of up to FEW lanes, and
// all behind the first TURNS, add lane by lane.
template <int M, int FEW = 0, int TURNS = 64, typename Flush>
__device__ __forceinline__ void wave_add_by_key(int key, const long long (&v)[M], Flush flush)
{
    const int lane = (int)(threadIdx.x & 63);
    unsigned long long pending = __ballot(key >= 0);
    for (int turn = 0; pending; ++turn) {
        if (TURNS < 64 && turn == TURNS) {
            if (pending >> lane & 1ull) flush(key, v);
            return;
        }
        const int leader = __ffsll(pending) - 1;
        const int k = __shfl(key, leader, 64);
        const bool mine = key == k;
        const unsigned long long grp = __ballot(mine);
        pending &= ~grp;
        if (FEW > 0 && __popcll(grp) <= FEW) {
            if (mine) flush(k, v);
            continue;
        }
        long long sum[M];
#pragma unroll
        for (int j = 0; j < M; ++j) sum[j] = wave_sum_i64(mine ? v[j] : 0ll);
        if (lane == leader) flush(k, sum);
    }
}

// ---- bubble statistics of a run --------------------------------------------------------------------
__device__ __forceinline__ int min_image_i(int d, int n)
{
    const int h = n / 2;
    int r = (d + h) % n;
    if (r < 0) r += n;
    return r - h;
}

// Node count of the `len` nodes from (x, y, z) on along x, and the sums of their integer
// minimal-image offsets from the anchor: along x the offsets rise by one from node to node and
// fall back to -floor(nx / 2) after the largest.
__device__ __forceinline__ void run_stats(int x, int y, int z, int len, const int32_t* anchor,
                                          const FieldArgs& a, long long v[4])
{
    const int d0 = min_image_i(x - anchor[0], a.nx), h = a.nx / 2;
    const long long m1 = min(len, a.nx - h - d0), m2 = len - m1;
    v[0] = len;
    v[1] = m1 * d0 + m1 * (m1 - 1) / 2 - m2 * h + m2 * (m2 - 1) / 2;
    v[2] = (long long)len * min_image_i(y - anchor[1], a.ny);
    v[3] = (long long)len * min_image_i(z - anchor[2], a.nz);
}

// Adds the runs of one word a lane (A: 0 for none) to their bubbles' counters; slot(s) is the bubble
// of the run that starts at bit s, or negative.  FEW and TURNS as above: in a box of many small
// bubbles that one block goes through, the chain is all (128^2 with 102 bubbles, a pass 235 us with
// every key in turn, 181 with 4 and 4, 201 with 1 and 8); large boxes hold few bubbles a wave, and
// their atomics count (512 x 512 x 256, 300 bubbles of R = 25: 1,915, 2,025, 1,880 us).
template <int FEW, int TURNS, typename F>
__device__ __forceinline__ void word_stats(uint64_t A, const Seg& g, const int32_t* anchors,
                                           unsigned long long* count, unsigned long long* sums,
                                           const FieldArgs& a, F slot)
{
    while (__ballot(A != 0ull)) {  // every lane stays for the aggregation
        int b = -1;
        long long v[4] = {0, 0, 0, 0};
        if (A) {
            const int s = __ffsll((long long)A) - 1;
            const uint64_t run = run_at(A, s);
            A &= ~run;
            b = slot(s);
            if (b >= 0) run_stats(g.x0 + s, g.y, g.z, __popcll(run), anchors + 3 * b, a, v);
        }
        // two's-complement wrap-around makes unsigned adds exact signed sums
        wave_add_by_key<4, FEW, TURNS>(b, v, [&](int k, const long long* s) {
            const size_t o = (size_t)k * kStatStride;
            atomicAdd(count + o, (unsigned long long)s[0]);
            atomicAdd(sums + o + 0, (unsigned long long)s[1]);
            atomicAdd(sums + o + 1, (unsigned long long)s[2]);
            atomicAdd(sums + o + 2, (unsigned long long)s[3]);
        });
    }
}

}  // namespace sc
