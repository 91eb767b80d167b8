// sc_test.hip -- 2D output fields, FP64 EOS / Laplacian / totals, bubble statistics, merge
// criterion and blowing-agent source of libsc (gfx950); the gas mask and labels are in
// sc_label.hip, the 3D fields in sc_fields.hip.
//
// Every kernel reads the pull-layout populations: f_i(x, t) = stored_i(x - e_i) + w_i rho_ref.
#include <algorithm>

#include "sc_device.hpp"
#include "sc_internal.hpp"
#include "sc_runs.hpp"

namespace sc {

static dim3 grid_for(int64_t n)
{
    int64_t b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    return dim3((unsigned)b);
}

// Coordinates of node n.  n < N <= 2^31 (sc_create bounds a population array to 2^32 bytes), so
// 32-bit unsigned division is exact, at a fraction of the cost of 64-bit division.
__device__ __forceinline__ void coords3(int64_t n, int nx, int ny, int& x, int& y, int& z)
{
    const uint32_t m = (uint32_t)n;
    const uint32_t r = m / (uint32_t)nx;
    x = (int)(m - r * (uint32_t)nx);
    y = (int)(r % (uint32_t)ny);
    z = (int)(r / (uint32_t)ny);
}

__device__ __forceinline__ int64_t idx3(int x, int y, int z, int nx, int ny)
{
    return (int64_t)x + (int64_t)nx * ((int64_t)y + (int64_t)ny * z);
}

// Node x + s * e_i (s = +1 downstream, -1 upstream), periodic.
template <int Q>
__device__ __forceinline__ int64_t shifted(int x, int y, int z, int i, int s, const FieldArgs& a)
{
    using L = lat<Q>;
    return idx3(wrap_once(x + s * L::ex[i], a.nx), wrap_once(y + s * L::ey[i], a.ny),
                wrap_once(z + s * L::ez[i], a.nz), a.nx, a.ny);
}

// FP32 deviation sum of node n (the same order as the step kernel).
template <int Q, typename S>
__device__ __forceinline__ float dev_sum_f(const S* f, int64_t n, const FieldArgs& a, float* g)
{
    int x, y, z;
    coords3(n, a.nx, a.ny, x, y, z);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        g[i] = load_f(f[(int64_t)i * a.N + shifted<Q>(x, y, z, i, -1, a)]);
        s += g[i];
    }
    return s;
}

// Sum of the stored deviations of node n, in double.
template <int Q, typename S>
__device__ __forceinline__ double dev_d(const S* f, int64_t n, const FieldArgs& a)
{
    int x, y, z;
    coords3(n, a.nx, a.ny, x, y, z);
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i)
        s += (double)load_f(f[(int64_t)i * a.N + shifted<Q>(x, y, z, i, -1, a)]);
    return s;
}

// FP64 density of node n: rho_ref + sum of the stored deviations.
template <int Q, typename S>
__device__ __forceinline__ double rho_d(const S* f, int64_t n, const FieldArgs& a)
{
    return a.rho_ref_d + dev_d<Q, S>(f, n, a);
}

// EOS pressure at node n: one component, p = rho/3 + (G/6) psi^2; two components (the gas
// component in a.f2, same storage, shifted by a.rho_ref2), p = (rho_l + rho_v)/3 + (Gx/3) rho_l rho_v.
template <int Q, typename S>
__device__ __forceinline__ double pressure_at(const S* f, int64_t n, const FieldArgs& a)
{
    const double r = rho_d<Q, S>(f, n, a);
    if (a.f2) {
        const double rv = a.rho_ref2 + dev_d<Q, S>((const S*)a.f2, n, a);
        return (r + rv) / 3.0 + (a.Gx / 3.0) * r * rv;
    }
    return pressure_d(r, a.Gd);
}

// ---- psi and the reported fields (FP64 arithmetic, FP32 output) -------------------------------
template <int Q, typename S>
__global__ void k_psi(const S* f, double* psi, FieldArgs a)
{
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N;
         n += (int64_t)gridDim.x * blockDim.x)
        psi[n] = psi_f(rho_d<Q, S>(f, n, a));
}

// rho and u = (j + F/2)/rho with the Shan-Chen force of the current state.
template <int Q, typename S>
__global__ void k_fields(const S* f, const double* psi, float* rho_out, float* u_out, FieldArgs a)
{
    using L = lat<Q>;
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N;
         n += (int64_t)gridDim.x * blockDim.x) {
        int x, y, z;
        coords3(n, a.nx, a.ny, x, y, z);
        double g[Q];
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            g[i] = (double)load_f(f[(int64_t)i * a.N + shifted<Q>(x, y, z, i, -1, a)]);
            s += g[i];
        }
        const double rho = a.rho_ref_d + s;
        if (rho_out) rho_out[n] = (float)rho;
        if (!u_out) continue;
        double j[3] = {0.0, 0.0, 0.0}, F[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            j[0] += g[i] * L::ex[i];
            j[1] += g[i] * L::ey[i];
            j[2] += g[i] * L::ez[i];
        }
        const uint16_t oc = a.owner ? a.owner[n] : (uint16_t)0;
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const int64_t m = shifted<Q>(x, y, z, i, +1, a);
            double pn = psi[m];
            // barrier: a neighbour of another, un-merged bubble is seen as bulk liquid
            if (oc != 0) {
                const uint16_t on = a.owner[m];
                if (on != 0 && on != oc) pn = a.psi_ld;
            }
            F[0] += L::wd[i] * pn * L::ex[i];
            F[1] += L::wd[i] * pn * L::ey[i];
            F[2] += L::wd[i] * pn * L::ez[i];
        }
        const double pc = psi[n];
        for (int c = 0; c < L::d; ++c) {
            double Fc = -a.Gd * pc * F[c];
            if (a.grav) Fc += (rho - a.rho0d) * a.gd[c];  // gravity body force
            u_out[(int64_t)c * a.N + n] = (float)((j[c] + 0.5 * Fc) / rho);
        }
    }
}

// ---- FP64 EOS and its lattice Laplacian (Sec. 3.1, the criterion's operator) ----------------
template <int Q, typename S>
__global__ void k_pressure(const S* f, double* p, FieldArgs a)
{
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N;
         n += (int64_t)gridDim.x * blockDim.x)
        p[n] = pressure_at<Q, S>(f, n, a);
}

template <int Q>
__global__ void k_laplacian(const double* p, double* lap, FieldArgs a)
{
    using L = lat<Q>;
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N;
         n += (int64_t)gridDim.x * blockDim.x) {
        int x, y, z;
        coords3(n, a.nx, a.ny, x, y, z);
        const double pc = p[n];
        double acc = 0.0;
#pragma unroll
        for (int i = 1; i < Q; ++i) acc += L::wd[i] * (p[shifted<Q>(x, y, z, i, +1, a)] - pc);
        lap[n] = 6.0 * acc;
    }
}

// ---- FP64 totals: wave64 shuffles -> LDS -> one partial per block -> fixed-order final sum ---
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Sums the stored values directly (a permutation of the pulled ones): M = N rho_ref + sum g,
// J = sum_i e_i sum_y g_i(y).
template <int Q, typename S>
__global__ void __launch_bounds__(256) k_totals(const S* f, double* partials, FieldArgs a)
{
    using L = lat<Q>;
    double m = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N;
         n += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const double g = (double)load_f(f[(int64_t)i * a.N + n]);
            m += g;
            jx += g * L::ex[i];
            jy += g * L::ey[i];
            jz += g * L::ez[i];
        }
    }
    __shared__ double red[4][4];
    m = wave_sum(m); jx = wave_sum(jx); jy = wave_sum(jy); jz = wave_sum(jz);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) { red[w][0] = m; red[w][1] = jx; red[w][2] = jy; red[w][3] = jz; }
    __syncthreads();
    if (threadIdx.x < 4) {
        double s = 0.0;
        for (int k = 0; k < 4; ++k) s += red[k][threadIdx.x];
        partials[(int64_t)blockIdx.x * 4 + threadIdx.x] = s;
    }
}

// ---- bubble statistics ------------------------------------------------------------------------
// One mask word a thread, its runs at once: 256^3 with 1.45 M gas nodes in 200 bubbles 171 us with a
// node a thread, whose 200,000 atomics met on 200 lines; 19 now.
__global__ void __launch_bounds__(256) k_stats(const uint32_t* __restrict__ labels,
                                               const uint64_t* __restrict__ mask,
                                               const int32_t* __restrict__ slot_of_root,
                                               const int32_t* __restrict__ anchors,
                                               unsigned long long* count,
                                               unsigned long long* sums, int64_t words, FieldArgs a)
{
    const int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const uint64_t A = w < words ? mask[w] : 0ull;
    if (!__ballot(A != 0ull)) return;
    const Seg g = seg_of(w < words ? w : 0, a);
    word_stats<1, 8>(A, g, anchors, count, sums, a,
               [&](int s) { return slot_of_root[labels[g.n + s] - 1]; });
}

// Gas-node list of the fed bubbles, in node order, without a global atomic per node or per wave:
// every block owns a contiguous chunk of nodes; the blocks count their fed gas nodes, one wave
// turns the counts into offsets, and each block writes its nodes from its offset on.
constexpr int kListBlocks = 1024;

static int64_t list_chunk(int64_t N)
{
    return ((N + (int64_t)kListBlocks * 256 - 1) / ((int64_t)kListBlocks * 256)) * 256;
}

__device__ __forceinline__ bool fed_gas(const uint32_t* labels, const int32_t* slot_of_root,
                                        const int32_t* feed, int64_t n, int64_t N, int& b)
{
    b = -1;
    if (n >= N) return false;
    const uint32_t L = labels[n];
    if (!L) return false;
    const int s = slot_of_root[L - 1];
    if (s < 0 || !feed[s]) return false;
    b = s;
    return true;
}

__global__ void __launch_bounds__(256) k_gas_count(const uint32_t* labels,
                                                   const int32_t* slot_of_root,
                                                   const int32_t* feed, unsigned int* counts,
                                                   int64_t N, int64_t chunk)
{
    const int64_t begin = blockIdx.x * chunk;
    unsigned int c = 0;
    for (int64_t n0 = begin; n0 < begin + chunk && n0 < N; n0 += 256) {
        int b;
        c += (unsigned int)__syncthreads_count(
            fed_gas(labels, slot_of_root, feed, n0 + threadIdx.x, N, b));
    }
    if (threadIdx.x == 0) counts[blockIdx.x] = c;
}

// One wave: exclusive prefix sums of the block counts in place, and their total.
__global__ void __launch_bounds__(64) k_gas_scan(unsigned int* counts, int n, unsigned int* total)
{
    const int lane = (int)threadIdx.x;
    unsigned int carry = 0;
    for (int c0 = 0; c0 < n; c0 += 64) {
        const int i = c0 + lane;
        const unsigned int v = i < n ? counts[i] : 0u;
        unsigned int x = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned int y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (i < n) counts[i] = carry + x - v;
        carry += __shfl(x, 63, 64);
    }
    if (lane == 0) *total = carry;
}

__global__ void __launch_bounds__(256) k_gas_write(const uint32_t* labels,
                                                   const int32_t* slot_of_root,
                                                   const int32_t* feed,
                                                   const unsigned int* offsets,
                                                   uint32_t* list_node, int32_t* list_slot,
                                                   int64_t N, int64_t chunk)
{
    __shared__ unsigned int wcnt[4];
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    unsigned int base = offsets[blockIdx.x];
    const int64_t begin = blockIdx.x * chunk;
    for (int64_t n0 = begin; n0 < begin + chunk && n0 < N; n0 += 256) {
        const int64_t n = n0 + threadIdx.x;
        int b;
        const bool g = fed_gas(labels, slot_of_root, feed, n, N, b);
        const unsigned long long m = __ballot(g);
        if (lane == 0) wcnt[w] = (unsigned int)__popcll(m);
        __syncthreads();
        unsigned int off = base;
        for (int k = 0; k < w; ++k) off += wcnt[k];
        const unsigned int tot = wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
        if (g) {
            const unsigned int k = off + (unsigned int)__popcll(m & below);
            list_node[k] = (uint32_t)n;
            list_slot[k] = b;
        }
        base += tot;
        __syncthreads();  // wcnt is rewritten by the next pass
    }
}

// ---- merge criterion (Sec. 3.1 eta_m, Sec. 4): one thread per candidate pair -----------------
template <int Q>
__device__ __forceinline__ int64_t walk_node(const MergePair& pr, int k, const FieldArgs& a)
{
#pragma clang fp contract(off)
    double pt[3];
    for (int c = 0; c < 3; ++c) pt[c] = pr.cen_a[c] + pr.dv[c] * (double)k / (double)pr.T;
    int x = (int)floor(pt[0] + 0.5) % a.nx; if (x < 0) x += a.nx;
    int y = (int)floor(pt[1] + 0.5) % a.ny; if (y < 0) y += a.ny;
    int z = 0;
    if (lat<Q>::d == 3) { z = (int)floor(pt[2] + 0.5) % a.nz; if (z < 0) z += a.nz; }
    return idx3(x, y, z, a.nx, a.ny);
}

// One wave tests one pair: the lanes take consecutive samples of the walk, so the walk's node
// arithmetic and label loads run side by side instead of one after another.  Repeats of the
// previous sample's node are dropped and positions counted over the kept samples, exactly as a
// sequential walk would; the densest film node is the first of the maxima in walk order, and the
// Laplacian's terms are summed by lane 0 in direction order.  Every lane of the wave must call
// this; all of them return the same result.
__device__ __forceinline__ int wave_max_i(int v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}
__device__ __forceinline__ int wave_min_i(int v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
    return v;
}
__device__ __forceinline__ double wave_max_d(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

template <int Q, typename S>
__device__ MergeResult merge_pair_wave(const MergePair& pr, const uint32_t* labels, const S* f,
                                       int film_max, const FieldArgs& a)
{
    using L = lat<Q>;
    const int lane = (int)(threadIdx.x & 63);
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int nk = pr.T + 1;
    MergeResult r;
    r.fired = 0; r.film_len = -1; r.film_node = -1; r.lap_p = 0.0; r.rho_film = 0.0;
    // Visits the kept samples chunk by chunk: fn(kept, pos, node) per lane, with the chunk's
    // lanes in walk order; fn returns false (wave-uniformly) to stop.
    auto walk = [&](auto fn) {
        int64_t carry_node = -1;
        int carry_pos = -1;
        for (int k0 = 0; k0 < nk; k0 += 64) {
            const int k = k0 + lane;
            const bool in = k < nk;
            const int64_t nd = in ? walk_node<Q>(pr, k, a) : (int64_t)-2;
            int64_t prev = __shfl_up(nd, 1, 64);
            if (lane == 0) prev = carry_node;
            const bool keep = in && nd != prev;
            const unsigned long long km = __ballot(keep);
            const int pos = carry_pos + __popcll(km & below) + 1;
            if (!fn(keep, pos, nd)) return;
            carry_pos += __popcll(km);
            const int last = min(63, nk - 1 - k0);
            carry_node = __shfl(nd, last, 64);
        }
    };
    // last node of a; then the first node of b after it
    int sa = -1;
    walk([&](bool keep, int pos, int64_t nd) {
        const int c = (keep && labels[nd] == pr.label_a) ? pos : -1;
        sa = max(sa, wave_max_i(c));
        return true;
    });
    if (sa < 0) return r;
    int sb = -1;
    walk([&](bool keep, int pos, int64_t nd) {
        const int c = (keep && pos > sa && labels[nd] == pr.label_b) ? pos : 0x7fffffff;
        const int m = wave_min_i(c);
        if (m != 0x7fffffff) sb = m;
        return sb < 0;
    });
    const int len = sb - sa - 1;
    if (sb < 0 || len < 1 || len > film_max) return r;
    // film run: positions sa+1 .. sb-1; liquid only; densest node first on ties
    bool clean = true;
    int64_t cstar = -1;
    double best = 0.0;
    walk([&](bool keep, int pos, int64_t nd) {
        const bool film = keep && pos > sa && pos < sb;
        if (__ballot(film && labels[nd] != 0)) clean = false;
        const double rho = film ? rho_d<Q, S>(f, nd, a) : -INFINITY;
        const double m = wave_max_d(rho);
        const unsigned long long at = __ballot(film && rho == m);
        if (at) {
            const int l0 = __ffsll(at) - 1;
            const int64_t node = __shfl(nd, l0, 64);
            if (cstar < 0 || m > best) {
                cstar = node;
                best = m;
            }
        }
        return true;
    });
    if (!clean) return r;
    int x, y, z;
    coords3(cstar, a.nx, a.ny, x, y, z);
    const double pc = pressure_at<Q, S>(f, cstar, a);
    double term = 0.0;
    if (lane >= 1 && lane < Q) {
        const int64_t m = shifted<Q>(x, y, z, lane, +1, a);
        term = L::wd[lane] * (pressure_at<Q, S>(f, m, a) - pc);
    }
    double acc = 0.0;
    for (int i = 1; i < Q; ++i) acc += __shfl(term, i, 64);
    const double lap = 6.0 * acc;
    r.film_len = len;
    r.film_node = cstar;
    r.lap_p = lap;
    r.rho_film = best;
    r.fired = lap >= 0.0 ? 1 : 0;
    return r;
}

// One wave (one block of 64) per candidate pair, over the first min(*count_d, npairs) pairs.
template <int Q, typename S>
__global__ void __launch_bounds__(64) k_merge(const S* f, const uint32_t* labels,
                                              const MergePair* pairs, MergeResult* res,
                                              int npairs, const int32_t* count_d, int film_max,
                                              FieldArgs a)
{
    const int p = blockIdx.x;
    if (count_d && *count_d < npairs) npairs = *count_d;
    if (p >= npairs) return;
    const MergeResult r = merge_pair_wave<Q, S>(pairs[p], labels, f, film_max, a);
    if (threadIdx.x == 0) res[p] = r;
}

// ---- blowing-agent source (Sec. 3): f_i(x) += w_i dm_b / n_b on the gas nodes of bubble b ----
// Each step bubble b is owed T_b = owed_b + dm_b: what earlier steps could not place plus this
// step's release.  Every listed node adds w_i T_b / n_b to its populations and rounds the sum
// into the storage type: to nearest for FP32, stochastically for FP16/BF16, whose spacing at a
// gas node (~5e-4 at -0.59 in FP16) exceeds the per-step increment (~1e-7) by orders of
// magnitude, so rounding to nearest would drop every increment.  The exact gain of the stored
// values (FP64 differences) is summed per bubble in fixed point (2^-40 units, integer atomics,
// so the sum does not depend on the order of the nodes), and k_source_close then sets
// owed_b = T_b - gain_b: the ledger carries what the storage could not take into the next step.

// The storage value next to the 16-bit pattern b toward +inf (up) or -inf: sign-magnitude
// layout, so moving away from zero adds one to the magnitude; +-0 steps to +-the smallest
// subnormal.
__device__ __forceinline__ uint16_t next_bits16(uint16_t b, bool up)
{
    const bool neg = (b & 0x8000u) != 0;
    if ((b & 0x7fffu) == 0) return up ? 0x0001u : 0x8001u;
    return (up != neg) ? (uint16_t)(b + 1u) : (uint16_t)(b - 1u);
}

// v rounded into the storage type.  FP32: to nearest.  FP16 / BF16: stochastically, to one of
// the two storage values lo <= v <= hi, hi with probability (v - lo) / (hi - lo), u in [0, 1),
// so the expected stored value is v.  (S)(float)v is one of lo, hi even where rounding twice
// picks the farther one; which of them it is follows from comparing it with v.
template <typename S>
__device__ __forceinline__ S round_into(double v, double u)
{
    const S h = static_cast<S>(static_cast<float>(v));
    const double hd = (double)static_cast<float>(h);
    if (hd == v) return h;
    const bool below = hd < v;
    const S o = __builtin_bit_cast(S, next_bits16(__builtin_bit_cast(uint16_t, h), below));
    const double od = (double)static_cast<float>(o);
    const double lo = below ? hd : od, hi = below ? od : hd;
    const bool take_hi = u < (v - lo) / (hi - lo);
    return take_hi ? (below ? o : h) : (below ? h : o);
}
template <>
__device__ __forceinline__ float round_into<float>(double v, double) { return (float)v; }

template <int Q, typename S>
__global__ void k_source(S* f, const uint32_t* list_node, const int32_t* list_slot, int64_t count,
                         SourceLedger led, int64_t t, FieldArgs a)
{
    using L = lat<Q>;
    // block-uniform trip count, so every lane of a wave reaches the aggregation of the gains
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k0 = blockIdx.x * (int64_t)blockDim.x; k0 < count; k0 += stride) {
        const int64_t k = k0 + threadIdx.x;
        int b = -1;
        long long gfx[1] = {0};
        if (k < count) {
            b = list_slot[k];
            const double T = led.owed[b] + led.dm[b];
            if (T == 0.0) {
                b = -1;
            } else {
                const double ab = T / led.nodes[b];
                const int64_t n = list_node[k];
                int x, y, z;
                coords3(n, a.nx, a.ny, x, y, z);
                // population i streams into n from n - e_i: 32-bit offsets per axis (indexed by
                // e + 1), as in the step kernel
                const uint32_t nx = a.nx, plane = (uint32_t)a.nx * (uint32_t)a.ny;
                const uint32_t xo[3] = {(uint32_t)wrap_once(x + 1, a.nx), (uint32_t)x,
                                        (uint32_t)wrap_once(x - 1, a.nx)};
                const uint32_t yo[3] = {(uint32_t)wrap_once(y + 1, a.ny) * nx, (uint32_t)y * nx,
                                        (uint32_t)wrap_once(y - 1, a.ny) * nx};
                const uint32_t zo[3] = {(uint32_t)wrap_once(z + 1, a.nz) * plane,
                                        (uint32_t)z * plane,
                                        (uint32_t)wrap_once(z - 1, a.nz) * plane};
                // every population of the node is loaded before any is stored (the stores
                // would otherwise order each load behind the previous direction's store)
                S* slot[Q];
                S old[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    slot[i] = f + (int64_t)i * a.N +
                              (xo[L::ex[i] + 1] + yo[L::ey[i] + 1] + zo[L::ez[i] + 1]);
                    old[i] = *slot[i];
                }
                double gain = 0.0;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    const double oldd = (double)load_f(old[i]);
                    const double u = unit_noise(
                        led.key, ((uint64_t)t * (uint64_t)a.N + (uint64_t)n) * (uint64_t)Q +
                                     (uint64_t)i);
                    const S nw = round_into<S>(oldd + L::wd[i] * ab, u);
                    *slot[i] = nw;
                    gain += (double)load_f(nw) - oldd;
                }
                gfx[0] = (long long)rint(gain * kGainScale);
            }
        }
        wave_add_by_key<1>(b, gfx, [&](int kb, const long long* s) {
            atomicAdd(&led.gain[(size_t)kb * kLedgerGainStride], (unsigned long long)s[0]);
        });
    }
}

// The gas list as a map: 1 + bubble slot of a listed node, 0 elsewhere (16 bytes a thread).
__global__ void k_fed_clear(uint16_t* map, int64_t N)
{
    const int64_t words = N / 8;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < words;
         k += (int64_t)gridDim.x * blockDim.x)
        reinterpret_cast<uint4*>(map)[k] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == 0)
        for (int64_t n = words * 8 + threadIdx.x; n < N; n += blockDim.x) map[n] = 0;
}

__global__ void k_fed_map(uint16_t* map, const uint32_t* list_node, const int32_t* list_slot,
                          int64_t count)
{
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * blockDim.x)
        map[list_node[k]] = (uint16_t)(list_slot[k] + 1);
}

// Closes the step's ledger once every node has added: owed_b = T_b - gain_b, gains back to zero.
__global__ void __launch_bounds__(256) k_source_close(SourceLedger led)
{
    for (int b = threadIdx.x; b < led.nb; b += blockDim.x) {
        const long long g = (long long)led.gain[(size_t)b * kLedgerGainStride];
        const double T = led.owed[b] + led.dm[b];
        led.owed[b] = T - (double)g * kGainUnit;
        led.gain[(size_t)b * kLedgerGainStride] = 0ull;
    }
}

// ---- film geometry of a bubble pair (Sec. 3 film disc; Fig. 3) --------------------------------
// Node of sample k on the line shifted by off, and its rounded (unwrapped) position r.
template <int Q>
__device__ __forceinline__ int64_t film_node(const FilmArgs& g, const double off[3], int k,
                                             const FieldArgs& a, double r[3])
{
#pragma clang fp contract(off)
    for (int c = 0; c < 3; ++c) {
        const double q = g.cen[c] + off[c] + g.dv[c] * (double)k / (double)g.T;
        r[c] = floor(q + 0.5);
    }
    if (lat<Q>::d == 2) r[2] = 0.0;
    int x = (int)r[0] % a.nx; if (x < 0) x += a.nx;
    int y = (int)r[1] % a.ny; if (y < 0) y += a.ny;
    int z = 0;
    if (lat<Q>::d == 3) { z = (int)r[2] % a.nz; if (z < 0) z += a.nz; }
    return idx3(x, y, z, a.nx, a.ny);
}

// One thread per line (offset (i, j)); the centre line also measures h.  Three walks per line,
// consecutive repeats dropped: the last node of bubble a, the first node of b after it, then the
// run between (liquid only) and, on the centre line, the arc positions of the two crossings.
template <int Q, typename S>
__global__ void k_film(const S* f, const uint32_t* labels, FilmArgs g, FilmOut* out,
                       FieldArgs a)
{
#pragma clang fp contract(off)
    const int side = 2 * g.K + 1;
    const int nlines = g.dim == 3 ? side * side : side;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nlines;
         t += gridDim.x * blockDim.x) {
        const int i = t % side - g.K;
        const int j = g.dim == 3 ? t / side - g.K : 0;
        if (i * i + j * j > g.K * g.K) continue;
        double off[3], r[3];
        for (int c = 0; c < 3; ++c) off[c] = (double)i * g.n1[c] + (double)j * g.n2[c];
        int sa = -1, sb = -1, pos = -1;
        int64_t prev = -1;
        for (int k = 0; k <= g.T; ++k) {
            const int64_t nd = film_node<Q>(g, off, k, a, r);
            if (nd == prev) continue;
            prev = nd;
            ++pos;
            if (labels[nd] == g.label_a) sa = pos;
        }
        if (sa < 0) continue;
        prev = -1; pos = -1;
        for (int k = 0; k <= g.T && sb < 0; ++k) {
            const int64_t nd = film_node<Q>(g, off, k, a, r);
            if (nd == prev) continue;
            prev = nd;
            ++pos;
            if (pos > sa && labels[nd] == g.label_b) sb = pos;
        }
        const int len = sb >= 0 ? sb - sa - 1 : 0;
        if (len < 1 || len > g.film_max) continue;
        const bool centre = i == 0 && j == 0;
        bool clean = true;
        double arc = 0.0, sA = 0.0, sB = 0.0, rp[3] = {0.0, 0.0, 0.0}, rho_p = 0.0;
        prev = -1; pos = -1;
        for (int k = 0; k <= g.T && pos < sb; ++k) {
            const int64_t nd = film_node<Q>(g, off, k, a, r);
            if (nd == prev) continue;
            prev = nd;
            ++pos;
            if (pos > sa && pos < sb && labels[nd] != 0) clean = false;
            if (centre) {
                const double rho = rho_d<Q, S>(f, nd, a);
                if (pos >= 1) {
                    const double dx = r[0] - rp[0], dy = r[1] - rp[1], dz = r[2] - rp[2];
                    const double seg = sqrt(dx * dx + dy * dy + dz * dz);
                    if (pos == sa + 1) sA = arc + seg * (a.theta - rho_p) / (rho - rho_p);
                    if (pos == sb) sB = arc + seg * (rho_p - a.theta) / (rho_p - rho);
                    arc += seg;
                }
                rho_p = rho;
                for (int c = 0; c < 3; ++c) rp[c] = r[c];
            }
        }
        if (!clean) continue;
        atomicAdd(&out->count, 1u);
        if (centre) out->h = sB - sA;
    }
}

// ---- barrier owner field ---------------------------------------------------------------------
// Seed: a gas node of a bubble (a component holding nuclei) gets that bubble's owner id.
__global__ void k_owner_seed(const uint32_t* labels, const int32_t* slot_of_root,
                             const uint16_t* ids, int nb, uint16_t* owner, int64_t N)
{
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < N;
         n += (int64_t)gridDim.x * blockDim.x) {
        uint16_t o = 0;
        if (nb > 0) {
            const uint32_t l = labels[n];
            if (l != 0) {
                const int32_t b = slot_of_root[l - 1];
                if (b >= 0) o = ids[b];
            }
        }
        owner[n] = o;
    }
}

// One corona layer: a node nobody owns takes the smallest owner id among its lattice
// neighbours (the velocity set is symmetric, so x + e_i covers the same nodes as x - e_i).
template <int Q>
__global__ void k_owner_grow(const uint16_t* in, uint16_t* out, FieldArgs a)
{
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N;
         n += (int64_t)gridDim.x * blockDim.x) {
        uint16_t o = in[n];
        if (o == 0) {
            int x, y, z;
            coords3(n, a.nx, a.ny, x, y, z);
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const uint16_t v = in[shifted<Q>(x, y, z, i, +1, a)];
                if (v != 0 && (o == 0 || v < o)) o = v;
            }
        }
        out[n] = o;
    }
}

// Frontier nodes: owned nodes with a lattice neighbour owned by a different bubble (the only
// nodes whose force the barrier changes), appended in any order.
template <int Q>
__global__ void k_frontier_list(const uint16_t* owner, uint32_t* list, unsigned int* count,
                                FieldArgs a)
{
    for (int64_t n = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; n < a.N;
         n += (int64_t)gridDim.x * blockDim.x) {
        const uint16_t o = owner[n];
        if (o == 0) continue;
        int x, y, z;
        coords3(n, a.nx, a.ny, x, y, z);
        bool frontier = false;
#pragma unroll
        for (int i = 1; i < Q; ++i) {
            const uint16_t v = owner[shifted<Q>(x, y, z, i, +1, a)];
            if (v != 0 && v != o) frontier = true;
        }
        if (frontier) list[atomicAdd(count, 1u)] = (uint32_t)n;
    }
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n)
{
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x)
        p[k] = v;
}

// ---- launchers ------------------------------------------------------------------------------
#define SC_DISPATCH(q, storage, CALL)                                                             \
    do {                                                                                          \
        if (q == 9 && storage == SC_STORE_F32) { constexpr int QQ = 9; using SS = float; CALL; }  \
        else if (q == 9 && storage == SC_STORE_F16) { constexpr int QQ = 9; using SS = _Float16; CALL; } \
        else if (q == 9 && storage == SC_STORE_BF16) { constexpr int QQ = 9; using SS = __bf16; CALL; } \
        else if (q == 19 && storage == SC_STORE_F32) { constexpr int QQ = 19; using SS = float; CALL; } \
        else if (q == 19 && storage == SC_STORE_F16) { constexpr int QQ = 19; using SS = _Float16; CALL; } \
        else if (q == 19 && storage == SC_STORE_BF16) { constexpr int QQ = 19; using SS = __bf16; CALL; } \
        else return hipErrorInvalidValue;                                                         \
    } while (0)

hipError_t launch_psi(int storage, const void* f, double* psi, const FieldArgs& a, hipStream_t st)
{
    switch (storage) {
        case SC_STORE_F32:
            hipLaunchKernelGGL((k_psi<9, float>), grid_for(a.N), dim3(256), 0, st, (const float*)f,
                               psi, a);
            break;
        case SC_STORE_F16:
            hipLaunchKernelGGL((k_psi<9, _Float16>), grid_for(a.N), dim3(256), 0, st,
                               (const _Float16*)f, psi, a);
            break;
        case SC_STORE_BF16:
            hipLaunchKernelGGL((k_psi<9, __bf16>), grid_for(a.N), dim3(256), 0, st,
                               (const __bf16*)f, psi, a);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fields(int q, int storage, const void* f, const double* psi, float* rho,
                         float* u, const FieldArgs& a, hipStream_t st)
{
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_fields<QQ, SS>), grid_for(a.N), dim3(256), 0, st,
                                   (const SS*)f, psi, rho, u, a));
    return hipGetLastError();
}

hipError_t launch_pressure(int q, int storage, const void* f, double* p, const FieldArgs& a,
                           hipStream_t st)
{
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_pressure<QQ, SS>), grid_for(a.N), dim3(256), 0, st,
                                   (const SS*)f, p, a));
    return hipGetLastError();
}

hipError_t launch_laplacian(const double* p, double* lap, const FieldArgs& a, hipStream_t st)
{
    hipLaunchKernelGGL((k_laplacian<9>), grid_for(a.N), dim3(256), 0, st, p, lap, a);
    return hipGetLastError();
}

hipError_t launch_totals(int q, int storage, const void* f, double* partials, double* out_d,
                         const FieldArgs& a, hipStream_t st)
{
    const int nb = totals_blocks(a.N);
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_totals<QQ, SS>), dim3(nb), dim3(256), 0, st, (const SS*)f,
                                   partials, a));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_totals_final(partials, nb, out_d, (double)a.N * a.rho_ref_d, st);
}

hipError_t launch_stats(const uint32_t* labels, uint32_t* scratch, const int32_t* slot_of_root,
                        const int32_t* anchors_d, unsigned long long* count_d,
                        unsigned long long* sums_d, const FieldArgs& a, hipStream_t st)
{
    const int64_t words = (int64_t)segs_of(a.nx) * a.ny * a.nz, nb = (words + 255) / 256;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_stats, dim3((unsigned)nb), dim3(256), 0, st, labels,
                       scratch_of(scratch, a).words, slot_of_root, anchors_d, count_d, sums_d,
                       words, a);
    return hipGetLastError();
}

int gas_list_scratch_words() { return kListBlocks; }

hipError_t launch_gas_list(const uint32_t* labels, const int32_t* slot_of_root,
                           const int32_t* feed_d, uint32_t* list_node, int32_t* list_slot,
                           unsigned int* count_d, unsigned int* block_counts, int64_t N,
                           hipStream_t st)
{
    const int64_t chunk = list_chunk(N);
    hipLaunchKernelGGL(k_gas_count, dim3(kListBlocks), dim3(256), 0, st, labels, slot_of_root,
                       feed_d, block_counts, N, chunk);
    hipLaunchKernelGGL(k_gas_scan, dim3(1), dim3(64), 0, st, block_counts, kListBlocks, count_d);
    hipLaunchKernelGGL(k_gas_write, dim3(kListBlocks), dim3(256), 0, st, labels, slot_of_root,
                       feed_d, block_counts, list_node, list_slot, N, chunk);
    return hipGetLastError();
}

hipError_t launch_merge_counted(int q, int storage, const void* f, const uint32_t* labels,
                                const MergePair* pairs_d, MergeResult* res_d, int cap,
                                const int32_t* count_d, int film_max, const FieldArgs& a,
                                hipStream_t st)
{
    if (cap <= 0) return hipSuccess;
    const dim3 g((unsigned)cap);
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_merge<QQ, SS>), g, dim3(64), 0, st, (const SS*)f, labels,
                                   pairs_d, res_d, cap, count_d, film_max, a));
    return hipGetLastError();
}

// ---- read-back of a test pass ----------------------------------------------------------------
__device__ void stage_out_body(const StageOut& o)
{
    const int t = threadIdx.x;
    if (t < 4) o.dst_tot[t] = o.tot[t];
    if (t >= 4 && t < 8 && o.tot2) o.dst_tot[t] = o.tot2[t - 4];
    if (o.head && t < 16) o.dst_head[t] = o.head[t];
    for (int k = t; k < o.n; k += blockDim.x) {
        o.dst_comp[k] = o.comp[k];
        o.dst_count[k] = o.count[(size_t)k * kStatStride];
        o.dst_sums[3 * k + 0] = o.sums[(size_t)k * kStatStride + 0];
        o.dst_sums[3 * k + 1] = o.sums[(size_t)k * kStatStride + 1];
        o.dst_sums[3 * k + 2] = o.sums[(size_t)k * kStatStride + 2];
    }
    for (int k = t; k < o.ledger_nb; k += blockDim.x) o.dst_owed[k] = o.owed[k];
    for (int k = t; k < o.npairs; k += blockDim.x) {
        o.dst_pairs[k] = o.pairs[k];
        o.dst_ab[2 * k] = o.ab[2 * k];
        o.dst_ab[2 * k + 1] = o.ab[2 * k + 1];
        o.dst_res[k] = o.res[k];
    }
}

// ---- device bubble table and candidate pairs --------------------------------------------------
static size_t tab_align(size_t b) { return (b + 255) & ~size_t(255); }

size_t bubble_tab_bytes(int n)
{
    const size_t m = (size_t)(n > 0 ? n : 1);
    return tab_align(64) + tab_align(4 * m) * 4 + tab_align(12 * m) +
           tab_align(8 * kStatStride * m) + tab_align(24 * m) + tab_align(8 * m);
}

BubbleTab bubble_tab_view(void* base, int n)
{
    const size_t m = (size_t)(n > 0 ? n : 1);
    char* p = (char*)base;
    BubbleTab t;
    t.head = (int32_t*)p; p += tab_align(64);
    t.comp = (uint32_t*)p; p += tab_align(4 * m);
    t.distinct = (uint32_t*)p; p += tab_align(4 * m);
    t.lead = (int32_t*)p; p += tab_align(4 * m);
    t.first = (int32_t*)p; p += tab_align(4 * m);
    t.anchors = (int32_t*)p; p += tab_align(12 * m);
    t.count = (unsigned long long*)p; p += tab_align(8 * kStatStride * m);
    t.sums = t.count + 1;
    t.cen = (double*)p; p += tab_align(24 * m);
    t.rad = (double*)p;
    return t;
}

// One block.  A bubble is a distinct nonzero label held by a nucleus node; its slot is the rank
// of its label among them and its lead nucleus the smallest index holding it (both O(n^2 / 1024)
// comparisons, a few microseconds for hundreds of nuclei).
__device__ void bubble_table_body(const uint32_t* labels, const int64_t* nuc_node, int n, int64_t N,
                                  const BubbleTab& prev, const BubbleTab& t,
                                  int32_t* slot_of_root, int nx, int ny)
{
    __shared__ int nb;
    // the previous pass's bubbles leave the slot map first (prev: the same buffer laid out for
    // the nucleus count of that pass; its head is zero before the first pass)
    const int nb_prev = prev.head[0];
    for (int b = threadIdx.x; b < nb_prev; b += blockDim.x)
        slot_of_root[prev.distinct[b] - 1] = -1;
    __syncthreads();
    if (threadIdx.x == 0) nb = 0;
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const int64_t nd = nuc_node[k];
        t.comp[k] = (nd >= 0 && nd < N) ? labels[nd] : 0u;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const uint32_t c = t.comp[k];
        int first = c != 0u;
        for (int j = 0; j < k && first; ++j)
            if (t.comp[j] == c) first = 0;
        t.first[k] = first;
        if (first) atomicAdd(&nb, 1);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        if (!t.first[k]) continue;
        const uint32_t c = t.comp[k];
        int b = 0;
        for (int j = 0; j < n; ++j)
            if (t.first[j] && t.comp[j] < c) ++b;
        t.distinct[b] = c;
        t.lead[b] = k;
        const int64_t a0 = nuc_node[k];
        t.anchors[3 * b + 0] = (int32_t)(a0 % nx);
        t.anchors[3 * b + 1] = (int32_t)((a0 / nx) % ny);
        t.anchors[3 * b + 2] = (int32_t)(a0 / ((int64_t)nx * ny));
        t.count[(size_t)b * kStatStride] = 0ull;
        t.sums[(size_t)b * kStatStride + 0] = 0ull;
        t.sums[(size_t)b * kStatStride + 1] = 0ull;
        t.sums[(size_t)b * kStatStride + 2] = 0ull;
        slot_of_root[c - 1] = b;
    }
    if (threadIdx.x == 0) {
        t.head[0] = nb;
        t.head[1] = 0;
    }
}

__global__ void __launch_bounds__(1024) k_bubble_table(const uint32_t* labels,
                                                       const int64_t* nuc_node, int n, int64_t N,
                                                       BubbleTab prev, BubbleTab t,
                                                       int32_t* slot_of_root, int nx, int ny)
{
    bubble_table_body(labels, nuc_node, n, N, prev, t, slot_of_root, nx, ny);
}

hipError_t launch_bubble_table(const uint32_t* labels, const int64_t* nuc_node, int n,
                               const BubbleTab& prev, const BubbleTab& t, int32_t* slot_of_root,
                               const FieldArgs& a, hipStream_t st)
{
    hipLaunchKernelGGL(k_bubble_table, dim3(1), dim3(1024), 0, st, labels, nuc_node, n, a.N,
                       prev, t, slot_of_root, a.nx, a.ny);
    return hipGetLastError();
}

__device__ __forceinline__ double min_image_d(double d, int n)
{
#pragma clang fp contract(off)
    return d - n * floor(d / n + 0.5);
}

// One block: centroid = anchor + (sum of integer offsets) / n and the equal-area (2D) or
// equal-volume (3D) radius, in the host's operation order; then the candidate pairs.
__device__ void find_pairs(const BubbleTab& t, const int32_t* group, int dim, int film_max,
                           MergePair* pairs, int32_t* ab, int cap, int nx, int ny, int nz)
{
#pragma clang fp contract(off)
    const int nb = t.head[0];
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
        const double n = (double)t.count[(size_t)b * kStatStride];
        for (int c = 0; c < 3; ++c)
            t.cen[3 * b + c] = (double)t.anchors[3 * b + c] +
                               (double)(long long)t.sums[(size_t)b * kStatStride + c] / n;
        if (dim == 2) {
            t.cen[3 * b + 2] = 0.0;
            t.rad[b] = sqrt(n / M_PI);
        } else {
            t.rad[b] = cbrt(3.0 * n / (4.0 * M_PI));
        }
    }
    __syncthreads();
    const int64_t total = (int64_t)nb * nb;
    for (int64_t p = threadIdx.x; p < total; p += blockDim.x) {
        const int a = (int)(p / nb), b = (int)(p % nb);
        if (b <= a) continue;
        if (group[t.lead[a]] == group[t.lead[b]]) continue;
        double dv[3];
        dv[0] = min_image_d(t.cen[3 * b + 0] - t.cen[3 * a + 0], nx);
        dv[1] = min_image_d(t.cen[3 * b + 1] - t.cen[3 * a + 1], ny);
        dv[2] = (dim == 3) ? min_image_d(t.cen[3 * b + 2] - t.cen[3 * a + 2], nz) : 0.0;
        const double dist = sqrt(dv[0] * dv[0] + dv[1] * dv[1] + dv[2] * dv[2]);
        if (dist > t.rad[a] + t.rad[b] + (double)film_max + 1e-6) continue;
        const int T = (int)ceil(dist);
        if (T <= 0) continue;
        const int k = atomicAdd(&t.head[1], 1);
        if (k >= cap) continue;
        MergePair mp;
        for (int c = 0; c < 3; ++c) {
            mp.cen_a[c] = t.cen[3 * a + c];
            mp.dv[c] = dv[c];
        }
        mp.label_a = t.distinct[a];
        mp.label_b = t.distinct[b];
        mp.T = T;
        mp.pad = 0;
        pairs[k] = mp;
        ab[2 * k] = a;
        ab[2 * k + 1] = b;
    }
}

__global__ void __launch_bounds__(1024) k_pairs(BubbleTab t, const int32_t* group, int dim,
                                                int film_max, MergePair* pairs, int32_t* ab,
                                                int cap, int nx, int ny, int nz)
{
    find_pairs(t, group, dim, film_max, pairs, ab, cap, nx, ny, nz);
}

hipError_t launch_pairs(const BubbleTab& t, const int32_t* group, int dim, int film_max,
                        MergePair* pairs, int32_t* ab, int cap, const FieldArgs& a,
                        hipStream_t st)
{
    hipLaunchKernelGGL(k_pairs, dim3(1), dim3(1024), 0, st, t, group, dim, film_max, pairs, ab,
                       cap, a.nx, a.ny, a.nz);
    return hipGetLastError();
}

// The tail of a test pass in one block: candidate pairs, their merge test (one wave per pair,
// sixteen at a time) and the read-back into pinned host memory.
template <int Q, typename S>
__device__ void pass_tail_body(const BubbleTab& t, const int32_t* group, int dim, int film_max,
                               MergePair* pairs, int32_t* ab, MergeResult* res, int cap,
                               int do_pairs, const StageOut& o, const S* f, const uint32_t* labels,
                               const FieldArgs& a)
{
    if (do_pairs) {
        find_pairs(t, group, dim, film_max, pairs, ab, cap, a.nx, a.ny, a.nz);
        __syncthreads();
        const int found = min(t.head[1], cap);
        const int w = (int)(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
        for (int p = w; p < found; p += nw) {
            const MergeResult r = merge_pair_wave<Q, S>(pairs[p], labels, f, film_max, a);
            if ((threadIdx.x & 63) == 0) res[p] = r;
        }
        __syncthreads();
    }
    stage_out_body(o);
}

template <int Q, typename S>
__global__ void __launch_bounds__(1024) k_pass_tail(BubbleTab t, const int32_t* group, int dim,
                                                    int film_max, MergePair* pairs, int32_t* ab,
                                                    MergeResult* res, int cap, int do_pairs,
                                                    StageOut o, const S* f,
                                                    const uint32_t* labels, FieldArgs a)
{
    pass_tail_body<Q, S>(t, group, dim, film_max, pairs, ab, res, cap, do_pairs, o, f, labels, a);
}

// The whole test pass of a small box behind its mask words, in one block: the totals' final sum,
// the labels (union-find over the runs in LDS, every link of the box), the bubble table, the
// statistics, the pairs and the read-back.  On such a box each of the seven kernels this replaces
// is a launch and a latency or two: 128^2 with two bubbles 28 us of kernels and seven gaps.
template <int Q, typename S>
__global__ void __launch_bounds__(1024) k_pass_small(uint32_t* scratch,
                                                     uint32_t* __restrict__ labels,
                                                     const double* __restrict__ partials, int nparts,
                                                     double* tot, double base_mass, SmallPass p,
                                                     const S* f, FieldArgs a)
{
    using R = RowLinks<Q>;
    extern __shared__ uint64_t bits[];  // [words], then the parents: 32 a word at most
    __shared__ double part[4 * kSmallParts];
    const int segs = segs_of(a.nx), words = segs * a.ny * a.nz, t = threadIdx.x;
    const int h = (min(a.nx, kSeg) + 1) / 2;  // parents a word
    uint32_t* const lp = reinterpret_cast<uint32_t*>(bits + words);
    const uint64_t* const mask = scratch_of(scratch, a).words;
    for (int k = t; k < 4 * nparts; k += 1024) part[k] = partials[k];
    for (int w = t; w < words; w += 1024) {
        const uint64_t A = mask[w];
        bits[w] = A;
        for (uint64_t left = A; left;) {
            const int s = __ffsll((long long)left) - 1;
            left &= ~run_at(A, s);
            lp[w * h + (s >> 1)] = (uint32_t)(w * h + (s >> 1));
        }
    }
    __syncthreads();
    if (t < 4) {  // the partials in block order (launch_totals_final: by lanes, other roundings)
        double s = 0.0;
        for (int b = 0; b < nparts; ++b) s += part[4 * b + t];
        tot[t] = t == 0 ? base_mass + s : s;
    }
    auto unite = [&](int wa, int sa, int wb, int sb) {
        union_unite(LdsParents{lp}, (uint32_t)(wa * h + (sa >> 1)), (uint32_t)(wb * h + (sb >> 1)));
    };
    for (int w = t; w < words; w += 1024) {
        const uint64_t A = bits[w];
        if (!A) continue;
        const Seg g = seg_of(w, a);
        const int seg = g.x0 / kSeg, row = w - seg, last = g.width - 1;
        const int sn = seg + 1 < segs ? seg + 1 : 0, sb = seg > 0 ? seg - 1 : segs - 1;
        const int lastb = min(kSeg, a.nx - sb * kSeg) - 1;
        const bool first_gas = A & 1ull, last_gas = A >> last & 1ull;
        if (last_gas && (bits[row + sn] & 1ull)) unite(w, run_start(A, last), row + sn, 0);
#pragma unroll
        for (int d = 0; d < R::n; ++d) {
            const int r2 = (wrap_once(g.y + R::dy[d], a.ny) +
                            a.ny * wrap_once(g.z + R::dz[d], a.nz)) * segs;
            touching_runs(A, bits[r2 + seg], A & ~(A << 1), R::wide[d],
                          [&](int x, int y) { unite(w, x, r2 + seg, y); });
            if (!R::wide[d]) continue;
            if (last_gas && (bits[r2 + sn] & 1ull)) unite(w, run_start(A, last), r2 + sn, 0);
            if (first_gas && (bits[r2 + sb] >> lastb & 1ull))
                unite(w, 0, r2 + sb, run_start(bits[r2 + sb], lastb));
        }
    }
    __syncthreads();
    // every run's parent becomes its root, then the label of its root (1 + the root's node): once a
    // run, the lanes only look it up
    for (int pass = 0; pass < 2; ++pass) {
        for (int w = t; w < words; w += 1024) {
            for (uint64_t left = bits[w]; left;) {
                const int s = __ffsll((long long)left) - 1;
                left &= ~run_at(bits[w], s);
                uint32_t* const e = lp + w * h + (s >> 1);
                if (pass == 0) {
                    union_settle(LdsParents{lp}, (uint32_t)(w * h + (s >> 1)));
                } else {
                    const int wr = (int)*e / h, b = 2 * ((int)*e - wr * h);
                    const uint64_t W = bits[wr], starts = W & ~(W << 1);
                    const int row = wr / segs;
                    *e = (uint32_t)(row * a.nx + (wr - row * segs) * kSeg + b +
                                    (int)(~(starts >> b) & 1ull)) + 1;
                }
            }
        }
        __syncthreads();
    }
    const int lane = t & 63;
    {
        int w = __builtin_amdgcn_readfirstlane(t >> 6);
        int row = w / segs, seg = w - row * segs;
        const int drow = 16 / segs, dseg = 16 - drow * segs;
        for (; w < words; w += 16) {
            const uint64_t A = bits[w];
            uint32_t v = 0u;
            if (A >> lane & 1ull) v = lp[w * h + (run_start(A, lane) >> 1)];
            if (seg * kSeg + lane < a.nx) labels[row * a.nx + seg * kSeg + lane] = v;
            row += drow;
            seg += dseg;
            if (seg >= segs) {
                seg -= segs;
                ++row;
            }
        }
    }
    __syncthreads();
    bubble_table_body(labels, p.nuc_node, p.n, a.N, p.prev, p.tab, p.slot_of_root, a.nx, a.ny);
    __syncthreads();
    for (int w0 = t - lane; w0 < words; w0 += 1024) {  // whole waves: the sums are by wave
        const int w = w0 + lane;
        const Seg g = seg_of(w < words ? w : 0, a);
        word_stats<4, 4>(w < words ? bits[w] : 0ull, g, p.tab.anchors, p.tab.count, p.tab.sums, a,
                   [&](int s) { return p.slot_of_root[labels[g.n + s] - 1]; });
    }
    __threadfence();  // the counters were summed past this CU's cache
    __syncthreads();
    pass_tail_body<Q, S>(p.tab, p.group, Q == 9 ? 2 : 3, p.film_max, p.pairs, p.ab, p.res, p.cap,
                         p.do_pairs, p.out, f, labels, a);
}

static size_t small_pass_lds(const FieldArgs& a)
{
    const size_t words = (size_t)segs_of(a.nx) * a.ny * a.nz, h = (size_t)(std::min(a.nx, kSeg) + 1) / 2;
    return words * 8 + words * h * 4;
}

bool small_pass_fits(const FieldArgs& a)
{
    // up to 2^15 nodes: beyond that one CU's share of the labels takes longer than the launches it
    // saves
    return a.N <= 1 << 15 && !a.f2 && small_pass_lds(a) <= (size_t)140 * 1024;
}

hipError_t launch_pass_small(int q, int storage, const void* f, uint32_t* scratch,
                             uint32_t* labels, const double* partials, double* tot,
                             const SmallPass& p, const FieldArgs& a, hipStream_t st)
{
    const int nb = totals_blocks(a.N);
    if (!small_pass_fits(a) || nb > kSmallParts) return hipErrorInvalidValue;
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_pass_small<QQ, SS>), dim3(1), dim3(1024), small_pass_lds(a),
                                   st, scratch, labels, partials, nb, tot,
                                   (double)a.N * a.rho_ref_d, p, (const SS*)f, a));
    return hipGetLastError();
}

hipError_t launch_pass_tail(int q, int storage, const BubbleTab& t, const int32_t* group,
                            int film_max, MergePair* pairs, int32_t* ab, MergeResult* res,
                            int cap, int do_pairs, const StageOut& o, const void* f,
                            const uint32_t* labels, const FieldArgs& a, hipStream_t st)
{
    const int dim = q == 9 ? 2 : 3;
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_pass_tail<QQ, SS>), dim3(1), dim3(1024), 0, st, t, group,
                                   dim, film_max, pairs, ab, res, cap, do_pairs, o,
                                   (const SS*)f, labels, a));
    return hipGetLastError();
}

hipError_t launch_source(int q, int storage, void* f, const uint32_t* list_node,
                         const int32_t* list_slot, int64_t count, const SourceLedger& led,
                         int64_t t, const FieldArgs& a, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_source<QQ, SS>), grid_for(count), dim3(256), 0, st, (SS*)f,
                                   list_node, list_slot, count, led, t, a));
    return launch_source_close(led, st);
}

hipError_t launch_source_close(const SourceLedger& led, hipStream_t st)
{
    hipLaunchKernelGGL(k_source_close, dim3(1), dim3(256), 0, st, led);
    return hipGetLastError();
}

hipError_t launch_fed_map(uint16_t* map, const uint32_t* list_node, const int32_t* list_slot,
                          int64_t count, int64_t N, hipStream_t st)
{
    hipLaunchKernelGGL(k_fed_clear, grid_for((N + 7) / 8), dim3(256), 0, st, map, N);
    hipLaunchKernelGGL(k_fed_map, grid_for(count), dim3(256), 0, st, map, list_node, list_slot,
                       count);
    return hipGetLastError();
}

hipError_t launch_owner_seed(const uint32_t* labels, const int32_t* slot_of_root,
                             const uint16_t* ids_d, int nb, uint16_t* owner, int64_t N,
                             hipStream_t st)
{
    hipLaunchKernelGGL(k_owner_seed, grid_for(N), dim3(256), 0, st, labels, slot_of_root, ids_d,
                       nb, owner, N);
    return hipGetLastError();
}

hipError_t launch_film(int q, int storage, const void* f, const uint32_t* labels,
                       const FilmArgs& g, FilmOut* out_d, const FieldArgs& a, hipStream_t st)
{
    const int side = 2 * g.K + 1;
    const int nlines = g.dim == 3 ? side * side : side;
    const dim3 grid((unsigned)std::max(1, std::min(1024, (nlines + 255) / 256)));
    SC_DISPATCH(q, storage,
                hipLaunchKernelGGL((k_film<QQ, SS>), grid, dim3(256), 0, st, (const SS*)f,
                                   labels, g, out_d, a));
    return hipGetLastError();
}

hipError_t launch_frontier_list(int q, const uint16_t* owner, uint32_t* list,
                                unsigned int* count_d, const FieldArgs& a, hipStream_t st)
{
    if (q == 9)
        hipLaunchKernelGGL((k_frontier_list<9>), grid_for(a.N), dim3(256), 0, st, owner, list,
                           count_d, a);
    else if (q == 19)
        hipLaunchKernelGGL((k_frontier_list<19>), grid_for(a.N), dim3(256), 0, st, owner, list,
                           count_d, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_owner_grow(int q, const uint16_t* in, uint16_t* out, const FieldArgs& a,
                             hipStream_t st)
{
    if (q == 9)
        hipLaunchKernelGGL((k_owner_grow<9>), grid_for(a.N), dim3(256), 0, st, in, out, a);
    else if (q == 19)
        hipLaunchKernelGGL((k_owner_grow<19>), grid_for(a.N), dim3(256), 0, st, in, out, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, grid_for(n), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

}  // namespace sc
