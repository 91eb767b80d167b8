// sc_label.hip -- gas mask, FP64 totals and canonical bubble labels of libsc (gfx950).
//
// Labels are 1 + the smallest linear index of a component (Fig. 1 step 7).  The mask is kept as
// one 64-bit word for each 64-node segment of a row along x, and the union-find works on the runs
// of a word instead of on nodes: a bubble of R = 12 has 7,200 nodes in about 450 runs, and all
// links between two rows are found with a few bit operations.  Only run starts have parents.  Two
// starts of a row are never neighbours unless a segment ends between them, so the parent of the
// start at column x of row r lies at entry r ceil(nx / 2) + x / 2, and the parents and the words
// together fit the N entries of the caller's scratch.
//   1. mask words (from a byte mask, from rho < threshold, or with the FP64 totals of the same
//      sweep);
//   2. k_label_local: a block unites the runs of its tile (16 x 16 rows of 64 nodes, in 2D 256
//      rows or 128) in LDS and writes every run's parent;
//   3. k_label_cross: the links between tiles, between segments and around the box, in global
//      memory;
//   4. k_label_flatten: every gas node takes its run's root.
// Roots link to the smaller index, so the labels are canonical whatever the order of the unions.
// 256^3 mask with 8.6% gas in 200 balls, microseconds with a union a node (local in 16^3 tiles) and
// now: mask 25 -> 6, local 118 -> 21, cross 268 -> 30, flatten 36 -> 36; the call 477 -> 111.
#include <algorithm>

#include "sc_device.hpp"
#include "sc_internal.hpp"
#include "sc_runs.hpp"
#include "sc_stepcore.hpp"

namespace sc {

namespace {

// Rows of a tile, and the lanes a word is split over in the two kernels that unite.  FINE: where the
// tiles do not fill the chip, its lanes would idle while one walks the up to 32 runs of a word of a
// fine mask (random masks, microseconds a call, a lane a word and so: 64^3 30% gas 250 -> 94, 1000^2
// 60% 218 -> 94); on large boxes the idle lanes of words with a run or two cost more than they give
// (256^3, 200 balls, lanes in the tiles and between them: 2 and 1 107 us, 2 and 2 110, 4 and 2 118,
// 4 and 8 133).
template <int Q, bool FINE>
struct LabelTile;
template <>
struct LabelTile<9, false> {
    static constexpr int RY = 256, RZ = 1, PARTS = 2, CROSS = 1;
};
template <>
struct LabelTile<9, true> {
    static constexpr int RY = 128, RZ = 1, PARTS = 8, CROSS = 8;
};
template <>
struct LabelTile<19, false> {
    static constexpr int RY = 16, RZ = 16, PARTS = 2, CROSS = 1;
};
template <>
struct LabelTile<19, true> {
    static constexpr int RY = 16, RZ = 16, PARTS = 4, CROSS = 8;
};

// ---- mask words ----------------------------------------------------------------------------------
// Rows of at most 32 nodes leave most of a wave idle if it takes them one by one, so NARROW packs as
// many as fit: the lanes of a wave are `rows` rows of 2^lg lanes.  Microseconds a call, one row and
// several a wave: 4 x 512 x 512 from the density 125 -> 46, from bytes (balls) 74 -> 43, test pass
// 133 -> 41; 16 x 256 x 256 55 -> 45, 58 -> 54, 53 -> 41.
struct Lanes {
    int lg, rows, sub, x;  // rows a wave takes at once, and this lane's row and column
};
template <bool NARROW>
__device__ __forceinline__ Lanes lanes_of(int nx)
{
    const int lane = (int)(threadIdx.x & 63);
    if (!NARROW) return Lanes{6, 1, 0, lane};
    const int lg = 32 - __clz(nx - 1);
    return Lanes{lg, kSeg >> lg, lane >> lg, lane & ((1 << lg) - 1)};
}
// The word of row `sub` out of a wave's ballot.
__device__ __forceinline__ uint64_t word_of_row(uint64_t ballot, int sub, int lg)
{
    return ballot >> (sub << lg) & below(1 << lg);
}

// A wave takes kMaskWords segments (or groups of rows) a turn, loads first.
constexpr int kMaskWords = 8;

template <bool NARROW>
__global__ void __launch_bounds__(256) k_mask_bytes(const uint8_t* __restrict__ mask,
                                                    uint64_t* __restrict__ out, int64_t words,
                                                    FieldArgs a)
{
    const int lane = (int)(threadIdx.x & 63);
    const Lanes ln = lanes_of<NARROW>(a.nx);
    const int64_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) + 4 * (int64_t)blockIdx.x;
    const int64_t step = kMaskWords * ln.rows;
    for (int64_t w0 = wave * step; w0 < words; w0 += 4 * (int64_t)gridDim.x * step) {
        bool gas[kMaskWords];
#pragma unroll
        for (int u = 0; u < kMaskWords; ++u) {
            gas[u] = false;
            const int64_t w = w0 + u * ln.rows + ln.sub;
            if (w >= words) continue;
            const Seg g = seg_of(w, a);
            if (ln.x < g.width) gas[u] = mask[g.n + ln.x] != 0;
        }
        uint64_t mine = 0ull;
#pragma unroll
        for (int u = 0; u < kMaskWords; ++u) {
            const uint64_t m = __ballot(gas[u]);
            if (NARROW) {
                const int64_t w = w0 + u * ln.rows + lane;
                if (lane < ln.rows && w < words) out[w] = word_of_row(m, lane, ln.lg);
            } else if (lane == u) {
                mine = m;
            }
        }
        if (!NARROW && lane < kMaskWords && w0 + lane < words) out[w0 + lane] = mine;
    }
}

// The same where every segment is full (nx a multiple of 64) and the mask 16-byte aligned: a lane
// takes 16 bytes, four lanes a word, a wave 16 words a turn.  16.8 MB: 25 us with a byte a lane,
// which a wave's 64-byte loads bound, 6 us so.
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v)
{
    return (v & 0xffu ? 1u : 0u) | (v & 0xff00u ? 2u : 0u) | (v & 0xff0000u ? 4u : 0u) |
           (v & 0xff000000u ? 8u : 0u);
}

__global__ void __launch_bounds__(256) k_mask_bytes16(const uint4* __restrict__ mask,
                                                      uint64_t* __restrict__ out, int64_t words)
{
    const int64_t quads = words * 4, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < quads; q += stride) {
        const uint4 v = mask[q];
        uint64_t m = (uint64_t)(nonzero_bytes(v.x) | nonzero_bytes(v.y) << 4 |
                                nonzero_bytes(v.z) << 8 | nonzero_bytes(v.w) << 12)
                     << 16 * (threadIdx.x & 3);
        // the four lanes of a word are all in range or all out of it
        m |= __shfl_xor((unsigned long long)m, 1, 64);
        m |= __shfl_xor((unsigned long long)m, 2, 64);
        if ((threadIdx.x & 3) == 0) out[q >> 2] = m;
    }
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// The gas mask rho < theta (FP64 density, the step kernel's order of the sum) and, with TOTALS, per
// block the sums of the pulled values and their momenta: the pulled values are a permutation of the
// stored ones, so these are the totals of the populations.  Two segments a turn, loads of both
// first (one wave carries many, and would otherwise wait out a full memory latency each).
template <int Q, typename S, bool TOTALS, bool NARROW>
__global__ void __launch_bounds__(256) k_mask_rho(const S* __restrict__ f,
                                                  uint64_t* __restrict__ out,
                                                  double* __restrict__ partials, int64_t words,
                                                  FieldArgs a)
{
    using L = lat<Q>;
    const int lane = (int)(threadIdx.x & 63);
    const int64_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) + 4 * (int64_t)blockIdx.x;
    double m = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
    const Lanes ln = lanes_of<NARROW>(a.nx);
    for (int64_t w0 = wave * 2 * ln.rows; w0 < words; w0 += 8 * (int64_t)gridDim.x * ln.rows) {
        float g[2][Q];
        bool on[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t w = w0 + u * ln.rows + ln.sub;
            on[u] = false;
            if (w >= words) continue;
            const Seg sg = seg_of(w, a);
            const int x = sg.x0 + ln.x, y = sg.y, z = sg.z;
            on[u] = ln.x < sg.width;
            if (on[u])
                pull_node<Q>(f, a.N, a.nx, a.ny, x, wrap_once(x - 1, a.nx), wrap_once(x + 1, a.nx),
                             y, wrap_once(y - 1, a.ny), wrap_once(y + 1, a.ny), z,
                             Q == 19 ? wrap_once(z - 1, a.nz) : 0,
                             Q == 19 ? wrap_once(z + 1, a.nz) : 0, g[u]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (w0 + u * ln.rows >= words) continue;
            bool gas = false;
            if (on[u]) {
                double s = 0.0, sx = 0.0, sy = 0.0, sz = 0.0;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const double v = (double)g[u][i];
                    s += v;
                    if (!TOTALS) continue;
                    if (L::ex[i] > 0) sx += v; else if (L::ex[i] < 0) sx -= v;
                    if (L::ey[i] > 0) sy += v; else if (L::ey[i] < 0) sy -= v;
                    if (L::ez[i] > 0) sz += v; else if (L::ez[i] < 0) sz -= v;
                }
                gas = a.rho_ref_d + s < a.theta;
                m += s;
                jx += sx;
                jy += sy;
                jz += sz;
            }
            const uint64_t mask = __ballot(gas);
            if (NARROW) {
                const int64_t w = w0 + u * ln.rows + lane;
                if (lane < ln.rows && w < words) out[w] = word_of_row(mask, lane, ln.lg);
            } else if (lane == 0) {
                out[w0 + u] = mask;
            }
        }
    }
    if constexpr (TOTALS) {
        __shared__ double red[4][4];
        m = wave_sum(m); jx = wave_sum(jx); jy = wave_sum(jy); jz = wave_sum(jz);
        const int w = threadIdx.x >> 6;
        if (lane == 0) { red[w][0] = m; red[w][1] = jx; red[w][2] = jy; red[w][3] = jz; }
        __syncthreads();
        if (threadIdx.x < 4) {
            double t = 0.0;
            for (int k = 0; k < 4; ++k) t += red[k][threadIdx.x];
            partials[(int64_t)blockIdx.x * 4 + threadIdx.x] = t;
        }
    }
}

// ---- union-find over runs, in global memory ---------------------------------------------------
// parent of a code (an agent-scope load: other blocks relink)
__device__ __forceinline__ uint32_t load_parent(const uint32_t* parent, uint32_t c)
{
    return __hip_atomic_load(parent + (c >> 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct GlobalParents {
    uint32_t* p;
    __device__ __forceinline__ uint32_t load(uint32_t c) const { return load_parent(p, c); }
    __device__ __forceinline__ void store(uint32_t c, uint32_t v) const
    {
        __hip_atomic_store(p + (c >> 1), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t min(uint32_t c, uint32_t v) const
    {
        return atomicMin(p + (c >> 1), v);
    }
};

// PARTS threads a word; the index of a run in LDS is its word's index times 32 plus half its first
// bit, which follows the global order, so a local root is the smallest node of its local set.
// Bound by the latency of the LDS chains.
template <int Q, bool FINE, typename T = LabelTile<Q, FINE>>
__global__ void __launch_bounds__(T::RY * T::RZ * T::PARTS)
k_label_local(uint32_t* scratch, uint32_t* zero_counter, FieldArgs a)
{
    using R = RowLinks<Q>;
    constexpr int kWords = T::RY * T::RZ;
    __shared__ uint64_t bits[kWords];
    __shared__ uint32_t lp[kWords * (kSeg / 2)];
    // the component counter of the flatten that follows starts at zero
    if (zero_counter && blockIdx.x == 0 && threadIdx.x == 0) *zero_counter = 0u;
    const LabelScratch sc = scratch_of(scratch, a);
    const int segs = segs_of(a.nx), gy = (a.ny + T::RY - 1) / T::RY;
    const int b = blockIdx.x, t = threadIdx.x / T::PARTS, part = threadIdx.x % T::PARTS;
    const int seg = b % segs, y0 = ((b / segs) % gy) * T::RY, z0 = (b / (segs * gy)) * T::RZ;
    const int iy = t % T::RY, iz = t / T::RY;
    const bool in = y0 + iy < a.ny && z0 + iz < a.nz;
    const uint32_t r = (uint32_t)(y0 + iy) + (uint32_t)a.ny * (uint32_t)(z0 + iz);
    const uint64_t A = in ? sc.words[(size_t)r * segs + seg] : 0ull;
    const uint64_t starts = run_starts<T::PARTS>(A, part);
    if (part == 0) bits[t] = A;
    for (uint64_t left = starts; left; left &= left - 1) {
        const int s = __ffsll((long long)left) - 1;
        lp[t * 32 + (s >> 1)] = (uint32_t)(t * 32 + (s >> 1));
    }
    if (!__syncthreads_or(A != 0ull)) return;
#pragma unroll
    for (int d = 0; d < R::n; ++d) {
        const int jy = iy + R::dy[d], jz = iz + R::dz[d];
        // a row outside the box has no bits, so only the tile's own edges need a test
        if (!starts || jy >= T::RY || jz < 0 || jz >= T::RZ) continue;
        const int u = jz * T::RY + jy;
        touching_runs(A, bits[u], starts, R::wide[d], [&](int sa, int sb) {
            union_unite(LdsParents{lp}, (uint32_t)(t * 32 + (sa >> 1)), (uint32_t)(u * 32 + (sb >> 1)));
        });
    }
    __syncthreads();
    for (uint64_t left = starts; left; left &= left - 1) {
        const int s = __ffsll((long long)left) - 1;
        const uint32_t e = union_root_halving(LdsParents{lp}, (uint32_t)(t * 32 + (s >> 1)));
        const int w = (int)(e >> 5), h = 2 * (int)(e & 31);
        // the start of the root's run is at bit h or h + 1 of its word: the one that is gas and
        // has no gas before it
        const uint64_t W = bits[w], first = W & ~(W << 1);
        const int x = seg * kSeg + h + (int)(~(first >> h) & 1ull);
        const uint32_t rr = (uint32_t)(y0 + w % T::RY) + (uint32_t)a.ny * (uint32_t)(z0 + w / T::RY);
        sc.parent[(size_t)r * sc.half + ((seg * kSeg + s) >> 1)] = code_of(rr, x, sc.half);
    }
}

// The links the tiles could not see, CROSS threads a word: to the next segment, to rows of other
// tiles, and around the box.  Bound by the latency of the parents' loads, which go past the L2s
// of the eight XCDs: both ends are followed together, and a pair of parents just united by this
// thread is not looked up again.
template <int Q, bool FINE>
__global__ void __launch_bounds__(256) k_label_cross(uint32_t* scratch, int64_t words, FieldArgs a)
{
    using T = LabelTile<Q, FINE>;
    using R = RowLinks<Q>;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, w = i / T::CROSS;
    if (w >= words) return;
    const int part = (int)(i % T::CROSS);
    const LabelScratch sc = scratch_of(scratch, a);
    const uint64_t A = sc.words[w];
    if (!A) return;
    const uint64_t starts = run_starts<T::CROSS>(A, part);
    const Seg g = seg_of(w, a);
    const uint32_t segs = (uint32_t)segs_of(a.nx), seg = (uint32_t)g.x0 / kSeg;
    const int last = g.width - 1;
    // the ends of the word: the first lane takes the links of both
    const bool first_gas = part == 0 && (A & 1ull), last_gas = part == 0 && (A >> last & 1ull);
    const uint32_t sn = seg + 1 < segs ? seg + 1 : 0, sb = seg > 0 ? seg - 1 : segs - 1;
    const int wb = min(kSeg, a.nx - (int)sb * kSeg);  // width of the segment before
    uint32_t la = 0u, lb = 0u;
    bool have = false;
    auto link = [&](uint32_t ra, int xa, uint32_t rb, int xb) {
        const uint32_t pa = load_parent(sc.parent, code_of(ra, xa, sc.half));
        const uint32_t pb = load_parent(sc.parent, code_of(rb, xb, sc.half));
        if (pa == pb || (have && pa == la && pb == lb)) return;
        la = pa;
        lb = pb;
        have = true;
        union_unite(GlobalParents{sc.parent}, pa, pb);
    };
    auto word = [&](uint32_t r, uint32_t s) { return sc.words[(size_t)r * segs + s]; };
    if (last_gas && (word(g.r, sn) & 1ull))
        link(g.r, g.x0 + run_start(A, last), g.r, (int)sn * kSeg);
#pragma unroll
    for (int d = 0; d < R::n; ++d) {
        const int y = g.y + R::dy[d], z = g.z + R::dz[d];
        const bool here = y < a.ny && z >= 0 && z < a.nz && y / T::RY == g.y / T::RY &&
                          z / T::RZ == g.z / T::RZ;
        if (here && !(R::wide[d] && (first_gas || last_gas))) continue;
        const uint32_t r2 = (uint32_t)wrap_once(y, a.ny) + (uint32_t)a.ny * (uint32_t)wrap_once(z, a.nz);
        if (!here)
            touching_runs(A, word(r2, seg), starts, R::wide[d],
                          [&](int sa, int sb2) { link(g.r, g.x0 + sa, r2, g.x0 + sb2); });
        if (!R::wide[d]) continue;
        if (last_gas && (word(r2, sn) & 1ull))
            link(g.r, g.x0 + run_start(A, last), r2, (int)sn * kSeg);
        if (first_gas) {
            const uint64_t B = word(r2, sb);
            if (B >> (wb - 1) & 1ull) link(g.r, g.x0, r2, (int)sb * kSeg + run_start(B, wb - 1));
        }
    }
}

// Blocks of k_label_flatten, at most: a block adds its components to the counter once, and those adds
// meet at one address, 4.4 ns each (4 x 512 x 512, 10% of single nodes: an add a wave of 16 nodes
// 290 us).
constexpr int kFlatBlocks = 2048;

// Labels from the words and the parents.  Bound by the write of the labels; most segments hold no
// gas and are filled with zeros at once, the others' walks to their roots go side by side.
template <int FW, bool NARROW>
__global__ void __launch_bounds__(256) k_label_flatten(uint32_t* __restrict__ lab,
                                                       uint32_t* scratch, uint32_t* ncomp,
                                                       int64_t words, FieldArgs a)
{
    const LabelScratch sc = scratch_of(scratch, a);
    const int lane = (int)(threadIdx.x & 63);
    const Lanes ln = lanes_of<NARROW>(a.nx);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6) + 4 * (int)blockIdx.x);
    const uint32_t segs = (uint32_t)segs_of(a.nx);
    unsigned roots = 0;
    const int64_t step = FW * ln.rows;
    for (int64_t w0 = (int64_t)wave * step; w0 < words; w0 += 4 * (int64_t)gridDim.x * step) {
        uint64_t A[FW];
        // row and first column of the segments, and where their labels start
        uint32_t row[FW];
        int x0[FW];
        bool any = false;
        if constexpr (NARROW) {  // a row a lane group: one segment each
#pragma unroll
            for (int u = 0; u < FW; ++u) {
                const int64_t w = w0 + u * ln.rows + ln.sub;
                A[u] = w < words ? sc.words[w] : 0ull;
                row[u] = (uint32_t)w;
                x0[u] = 0;
                any |= A[u] != 0ull;
            }
        } else {
#pragma unroll
            for (int u = 0; u < FW; ++u) A[u] = w0 + u < words ? sc.words[w0 + u] : 0ull;
#pragma unroll
            for (int u = 0; u < FW; ++u)  // the same in every lane: scalar, so that its tests are branches
                A[u] = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)A[u]) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(A[u] >> 32)) << 32;
            uint32_t rr = __builtin_amdgcn_readfirstlane((uint32_t)w0 / segs);
            uint32_t ss = (uint32_t)w0 - rr * segs;
#pragma unroll
            for (int u = 0; u < FW; ++u) {
                row[u] = rr;
                x0[u] = (int)ss * kSeg;
                if (++ss == segs) {
                    ss = 0;
                    ++rr;
                }
                any |= A[u] != 0ull;
            }
        }
        uint32_t v[FW];
#pragma unroll
        for (int u = 0; u < FW; ++u) v[u] = 0u;
        if (any) {
            uint32_t r[FW];
            int s[FW];
#pragma unroll
            for (int u = 0; u < FW; ++u) {
                r[u] = 0u;
                s[u] = 0;
                if (!A[u]) continue;
                s[u] = run_start(A[u], ln.x);
                r[u] = code_of(row[u], x0[u] + s[u], sc.half);
            }
            bool more = true;
            while (more) {
                more = false;
                uint32_t p[FW];
#pragma unroll
                for (int u = 0; u < FW; ++u) {
                    p[u] = r[u];
                    if (A[u] && (A[u] >> ln.x & 1ull)) p[u] = sc.parent[r[u] >> 1];
                }
#pragma unroll
                for (int u = 0; u < FW; ++u) {
                    more |= p[u] != r[u];
                    r[u] = p[u];
                }
            }
#pragma unroll
            for (int u = 0; u < FW; ++u) {
                if (!A[u] || !(A[u] >> ln.x & 1ull)) continue;
                v[u] = node_of_code(r[u], sc.half, a.nx) + 1;
                if (s[u] == ln.x && r[u] == code_of(row[u], x0[u] + ln.x, sc.half)) ++roots;
            }
        }
#pragma unroll
        for (int u = 0; u < FW; ++u)
            if (w0 + u * ln.rows + ln.sub < words && x0[u] + ln.x < a.nx)
                lab[(int64_t)row[u] * a.nx + x0[u] + ln.x] = v[u];
    }
    // one atomic a block that found any
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) roots += __shfl_xor(roots, off, 64);
    __shared__ unsigned found[4];
    if (lane == 0) found[threadIdx.x >> 6] = roots;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned n = found[0] + found[1] + found[2] + found[3];
        if (n) atomicAdd(ncomp, n);
    }
}

// Block partials to the totals, in a fixed order: a wave a component, every lane its partials in
// block order, then the lanes in a butterfly (25 us for 1,024 blocks as one chain of adds).
constexpr int kTotBlocks = 1024;

__global__ void __launch_bounds__(256) k_totals_final(const double* __restrict__ partials, int nb,
                                                      double* __restrict__ out, double base_mass)
{
    const int c = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double v[kTotBlocks / 64];
#pragma unroll
    for (int k = 0; k < kTotBlocks / 64; ++k)
        v[k] = lane + 64 * k < nb ? partials[(lane + 64 * k) * 4 + c] : 0.0;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kTotBlocks / 64; ++k) s += v[k];
    s = wave_sum(s);
    if (lane == 0) out[c] = (c == 0) ? base_mass + s : s;
}

bool narrow_rows(const FieldArgs& a) { return a.nx <= kSeg / 2; }
int rows_a_wave(const FieldArgs& a)  // as lanes_of
{
    int p = 1;
    while (p < a.nx && p < kSeg) p *= 2;
    return kSeg / p;
}

int64_t words_of(const FieldArgs& a) { return (int64_t)segs_of(a.nx) * a.ny * a.nz; }

dim3 word_grid(int64_t words, int per_block)
{
    const int64_t b = (words + per_block - 1) / per_block;
    return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 65536)));
}

template <int Q, typename S, bool TOTALS>
void mask_rho(const void* f, uint32_t* scratch, double* partials, int nb, const FieldArgs& a,
              hipStream_t st)
{
    if (narrow_rows(a))
        hipLaunchKernelGGL((k_mask_rho<Q, S, TOTALS, true>), dim3(nb), dim3(256), 0, st,
                           (const S*)f, scratch_of(scratch, a).words, partials, words_of(a), a);
    else
        hipLaunchKernelGGL((k_mask_rho<Q, S, TOTALS, false>), dim3(nb), dim3(256), 0, st,
                           (const S*)f, scratch_of(scratch, a).words, partials, words_of(a), a);
}

template <bool TOTALS>
hipError_t mask_rho_any(int q, int storage, const void* f, uint32_t* scratch, double* partials,
                        const FieldArgs& a, hipStream_t st)
{
    const int nb = totals_blocks(a.N);
    if (q == 9 && storage == SC_STORE_F32) mask_rho<9, float, TOTALS>(f, scratch, partials, nb, a, st);
    else if (q == 9 && storage == SC_STORE_F16) mask_rho<9, _Float16, TOTALS>(f, scratch, partials, nb, a, st);
    else if (q == 9 && storage == SC_STORE_BF16) mask_rho<9, __bf16, TOTALS>(f, scratch, partials, nb, a, st);
    else if (q == 19 && storage == SC_STORE_F32) mask_rho<19, float, TOTALS>(f, scratch, partials, nb, a, st);
    else if (q == 19 && storage == SC_STORE_F16) mask_rho<19, _Float16, TOTALS>(f, scratch, partials, nb, a, st);
    else if (q == 19 && storage == SC_STORE_BF16) mask_rho<19, __bf16, TOTALS>(f, scratch, partials, nb, a, st);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int Q, bool FINE>
int64_t label_tiles(const FieldArgs& a)
{
    using T = LabelTile<Q, FINE>;
    return (int64_t)segs_of(a.nx) * ((a.ny + T::RY - 1) / T::RY) * ((a.nz + T::RZ - 1) / T::RZ);
}

template <int Q, bool FINE>
hipError_t unite_words(uint32_t* scratch, uint32_t* ncomp, int64_t words, const FieldArgs& a,
                       hipStream_t st)
{
    using T = LabelTile<Q, FINE>;
    const int64_t tiles = label_tiles<Q, FINE>(a), cross = (words * T::CROSS + 255) / 256;
    if (tiles > 0x7fffffff || cross > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_label_local<Q, FINE>), dim3((unsigned)tiles),
                       dim3(T::RY * T::RZ * T::PARTS), 0, st, scratch, ncomp, a);
    hipLaunchKernelGGL((k_label_cross<Q, FINE>), dim3((unsigned)cross), dim3(256), 0, st, scratch,
                       words, a);
    return hipGetLastError();
}

template <int Q>
hipError_t label_words(uint32_t* lab, uint32_t* scratch, uint32_t* ncomp, const FieldArgs& a,
                       hipStream_t st)
{
    const int64_t words = words_of(a);
    const hipError_t e = label_tiles<Q, false>(a) <= 256
                             ? unite_words<Q, true>(scratch, ncomp, words, a, st)
                             : unite_words<Q, false>(scratch, ncomp, words, a, st);
    if (e != hipSuccess) return e;
    // one word a wave while the waves do not fill the chip (its latencies are then the bound); few
    // enough blocks that their counts do not queue at the one counter
    const bool narrow = narrow_rows(a);
    const int64_t turns = (words + rows_a_wave(a) - 1) / rows_a_wave(a);
    const int fw = turns < 16384 ? 1 : 4;
    const dim3 grid((unsigned)std::min<int64_t>((turns + 4 * fw - 1) / (4 * fw), kFlatBlocks)), block(256);
    if (narrow && fw == 1)
        hipLaunchKernelGGL((k_label_flatten<1, true>), grid, block, 0, st, lab, scratch, ncomp, words, a);
    else if (narrow)
        hipLaunchKernelGGL((k_label_flatten<4, true>), grid, block, 0, st, lab, scratch, ncomp, words, a);
    else if (fw == 1)
        hipLaunchKernelGGL((k_label_flatten<1, false>), grid, block, 0, st, lab, scratch, ncomp, words, a);
    else
        hipLaunchKernelGGL((k_label_flatten<4, false>), grid, block, 0, st, lab, scratch, ncomp, words, a);
    return hipGetLastError();
}

}  // namespace

int totals_blocks(int64_t N)
{
    const int64_t b = (N + 255) / 256;
    return (int)(b < kTotBlocks ? (b < 1 ? 1 : b) : kTotBlocks);
}

hipError_t launch_totals_final(const double* partials, int nb, double* out_d, double base_mass,
                               hipStream_t st)
{
    if (nb < 1 || nb > kTotBlocks) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_totals_final, dim3(1), dim3(256), 0, st, partials, nb, out_d, base_mass);
    return hipGetLastError();
}

hipError_t launch_mask_from_rho(int q, int storage, const void* f, uint32_t* scratch,
                                const FieldArgs& a, hipStream_t st)
{
    return mask_rho_any<false>(q, storage, f, scratch, nullptr, a, st);
}

hipError_t launch_mask_totals(int q, int storage, const void* f, uint32_t* scratch,
                              double* partials, double* out_d, const FieldArgs& a, hipStream_t st)
{
    const hipError_t e = mask_rho_any<true>(q, storage, f, scratch, partials, a, st);
    if (e != hipSuccess) return e;
    return launch_totals_final(partials, totals_blocks(a.N), out_d, (double)a.N * a.rho_ref_d, st);
}

hipError_t launch_mask_words(int q, int storage, const void* f, uint32_t* scratch,
                             double* partials, const FieldArgs& a, hipStream_t st)
{
    return mask_rho_any<true>(q, storage, f, scratch, partials, a, st);
}

hipError_t launch_mask_from_bytes(const uint8_t* mask_d, uint32_t* scratch, const FieldArgs& a,
                                  hipStream_t st)
{
    const int64_t words = words_of(a);
    if (a.nx % kSeg == 0 && (uintptr_t)mask_d % 16 == 0)
        hipLaunchKernelGGL(k_mask_bytes16, word_grid(words, 64), dim3(256), 0, st,
                           (const uint4*)mask_d, scratch_of(scratch, a).words, words);
    else if (narrow_rows(a))
        hipLaunchKernelGGL(k_mask_bytes<true>, word_grid(words, 4 * kMaskWords * rows_a_wave(a)),
                           dim3(256), 0, st, mask_d, scratch_of(scratch, a).words, words, a);
    else
        hipLaunchKernelGGL(k_mask_bytes<false>, word_grid(words, 4 * kMaskWords), dim3(256), 0, st,
                           mask_d, scratch_of(scratch, a).words, words, a);
    return hipGetLastError();
}

hipError_t launch_labels(int q, uint32_t* labels, uint32_t* scratch, uint32_t* ncomp_d,
                         const FieldArgs& a, hipStream_t st)
{
    if (q == 9) return label_words<9>(labels, scratch, ncomp_d, a, st);
    if (q == 19) return label_words<19>(labels, scratch, ncomp_d, a, st);
    return hipErrorInvalidValue;
}

}  // namespace sc
