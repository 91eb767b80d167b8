// sc_fields.hip -- reported fields and the pressure Laplacian of a D3Q19 box in one sweep (gfx950).
//
// Density and velocity, the mixture's fields, and p with its lattice Laplacian all form one FP64
// value a node (psi; both densities; p) and then combine it with the neighbours' values.  As two
// kernels over an N-sized FP64 array the populations were read twice (fields) and the value array
// written once and gathered 18 times.  Here a block owns a tile of a plane and marches in z, as
// the step does: the values of the tile and its one-node ring stay in LDS for three planes, a
// node's density and momentum in registers from its load until its output one plane later.
// Bound by HBM: the populations once (the ring's again from L2), the outputs once.  256^3, FP32
// storage, 1.54 GB each: rho and u 820 -> 338 us, p and its Laplacian 472 -> 335 us (4.6 TB/s, as
// fast as the marching step moves data).
#include <algorithm>

#include "sc_device.hpp"
#include "sc_internal.hpp"
#include "sc_stepcore.hpp"

namespace sc {

namespace {

enum { kFields = 0, kLaplacian = 1, kMixFields = 2 };

struct FieldOut {
    float *rho, *rho_v, *u;
    double *p, *lap;
};

// One component's density deviation and momentum of a node from its pulled values.
struct Moments {
    double s, j[3];
};
__device__ __forceinline__ Moments moments19(const float* g)
{
    using L = lat<19>;
    Moments m{0.0, {0.0, 0.0, 0.0}};
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const double v = (double)g[i];
        m.s += v;
        if (L::ex[i] > 0) m.j[0] += v; else if (L::ex[i] < 0) m.j[0] -= v;
        if (L::ey[i] > 0) m.j[1] += v; else if (L::ey[i] < 0) m.j[1] -= v;
        if (L::ez[i] > 0) m.j[2] += v; else if (L::ez[i] < 0) m.j[2] -= v;
    }
    return m;
}

// Up to 124 registers (the two load sets of a plane are in flight together): one block of 1024
// threads a CU.
template <typename S, int MODE>
__global__ void __launch_bounds__(1024) k_march3d(const S* __restrict__ f, FieldOut o, FieldArgs a,
                                                  int planes, StepGrid grid)
{
    using L = lat<19>;
    constexpr int V = MODE == kMixFields ? 2 : 1;  // values a node
    extern __shared__ double ring_lds[];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t N = a.N;
    const S* __restrict__ f2 = (const S*)a.f2;
    const int lb = logical_block(grid);
    const int bx = lb % grid.gx, by = (lb / grid.gx) % grid.gy, bz = lb / (grid.gx * grid.gy);
    const int t = threadIdx.x, tw = grid.tw, th = grid.th;
    const int pw = tw + 2, psz = pw * (th + 2);
    const int x0 = bx * tw, y0 = by * th, z0 = bz * planes;
    const int wx = min(tw, nx - x0), wy = min(th, ny - y0), ze = min(z0 + planes, nz);
    const int ty = t / tw, tx = t - ty * tw;
    const bool own = tx < wx && ty < wy;
    const int x = x0 + (own ? tx : 0), y = y0 + (own ? ty : 0);
    const int xm = wrap_once(x - 1, nx), xp = wrap_once(x + 1, nx);
    const int ym = wrap_once(y - 1, ny), yp = wrap_once(y + 1, ny);
    const bool ring = t < 2 * (wx + 2) + 2 * wy;
    int hlx, hly;
    ring_cell(t, wx, wy, hlx, hly);
    if (!ring) hlx = hly = 1;
    const int hx = wrap_once(x0 - 1 + hlx, nx), hy = wrap_once(y0 - 1 + hly, ny);
    const int hxm = wrap_once(hx - 1, nx), hxp = wrap_once(hx + 1, nx);
    const int hym = wrap_once(hy - 1, ny), hyp = wrap_once(hy + 1, ny);
    const int pc0 = pw * ((own ? ty : 0) + 1) + (own ? tx : 0) + 1;
    const int ph0 = pw * hly + hlx;
    double* const v0 = ring_lds;             // [4][th + 2][tw + 2]
    double* const v1 = ring_lds + 4 * psz;   // the mixture's gas density

    auto value = [&](double rl, double rv) -> double {
        if (MODE == kMixFields) return rl;
        if (MODE == kFields) return psi_f(rl);
        if (a.f2) return (rl + rv) / 3.0 + (a.Gx / 3.0) * rl * rv;
        return pressure_d(rl, a.Gd);
    };
    auto load = [&](int z, int k, Moments& ml, Moments& mv) {
        const int zm = wrap_once(z - 1, nz), zp = wrap_once(z + 1, nz);
        float g[19];
        if (own) {
            pull_plane<19>(f, N, nx, ny, x, xm, xp, y, ym, yp, z, zm, zp, g);
            ml = moments19(g);
            double rv = 0.0;
            if (MODE != kFields && f2) {
                pull_plane<19>(f2, N, nx, ny, x, xm, xp, y, ym, yp, z, zm, zp, g);
                mv = moments19(g);
                rv = a.rho_ref2 + mv.s;
            }
            v0[k * psz + pc0] = value(a.rho_ref_d + ml.s, rv);
            if (V == 2) v1[k * psz + pc0] = rv;
        }
        if (ring) {
            pull_plane<19>(f, N, nx, ny, hx, hxm, hxp, hy, hym, hyp, z, zm, zp, g);
            const double rl = a.rho_ref_d + sum_dev<19, double>(g);
            double rv = 0.0;
            if (MODE != kFields && f2) {
                pull_plane<19>(f2, N, nx, ny, hx, hxm, hxp, hy, hym, hyp, z, zm, zp, g);
                rv = a.rho_ref2 + sum_dev<19, double>(g);
            }
            v0[k * psz + ph0] = value(rl, rv);
            if (V == 2) v1[k * psz + ph0] = rv;
        }
    };

    Moments cl{}, cv{}, nl{}, nv{};
    load(wrap_once(z0 - 1, nz), 0, nl, nv);
    load(z0, 1, cl, cv);
    for (int z = z0; z < ze; ++z) {
        const int s = (z - z0 + 1) & 3, sn = (s + 1) & 3, sp = (s + 3) & 3;
        load(wrap_once(z + 1, nz), sn, nl, nv);
        __syncthreads();
        if (own) {
            const int64_t n = (int64_t)x + (int64_t)nx * ((int64_t)y + (int64_t)ny * z);
            auto near = [&](const double* v, int i) {
                const int slot = L::ez[i] > 0 ? sn : (L::ez[i] < 0 ? sp : s);
                return v[slot * psz + pc0 + L::ey[i] * pw + L::ex[i]];
            };
            const double vc = v0[s * psz + pc0];
            if (MODE == kLaplacian) {
                double acc = 0.0;
#pragma unroll
                for (int i = 1; i < 19; ++i) acc += L::wd[i] * (near(v0, i) - vc);
                if (o.p) o.p[n] = vc;
                if (o.lap) o.lap[n] = 6.0 * acc;
            } else if (MODE == kMixFields) {
                const double rl = vc, rv = v1[s * psz + pc0];
                if (o.rho) o.rho[n] = (float)rl;
                if (o.rho_v) o.rho_v[n] = (float)rv;
                if (o.u) {
                    double sx, sy, sz, wxx, wyy, wzz;
                    interaction_sum<19, double>([&](int i) { return near(v1, i); }, sx, sy, sz);
                    interaction_sum<19, double>([&](int i) { return near(v0, i); }, wxx, wyy, wzz);
                    const double Sf[3] = {rl * sx + rv * wxx, rl * sy + rv * wyy,
                                          rl * sz + rv * wzz};
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        o.u[(int64_t)c * N + n] =
                            (float)((cl.j[c] + cv.j[c] - 0.5 * a.Gx * Sf[c]) / (rl + rv));
                }
            } else {
                const double rho = a.rho_ref_d + cl.s;
                if (o.rho) o.rho[n] = (float)rho;
                const uint16_t oc = a.owner ? a.owner[n] : (uint16_t)0;
                double F[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int i = 1; i < 19; ++i) {
                    double pn = near(v0, i);
                    // barrier: a neighbour of another, un-merged bubble is seen as bulk liquid
                    if (oc != 0) {
                        const int64_t m =
                            (int64_t)(L::ex[i] > 0 ? xp : (L::ex[i] < 0 ? xm : x)) +
                            (int64_t)nx *
                                ((int64_t)(L::ey[i] > 0 ? yp : (L::ey[i] < 0 ? ym : y)) +
                                 (int64_t)ny * wrap_once(z + L::ez[i], nz));
                        const uint16_t on = a.owner[m];
                        if (on != 0 && on != oc) pn = a.psi_ld;
                    }
                    F[0] += L::wd[i] * pn * L::ex[i];
                    F[1] += L::wd[i] * pn * L::ey[i];
                    F[2] += L::wd[i] * pn * L::ez[i];
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double Fc = -a.Gd * vc * F[c];
                    if (a.grav) Fc += (rho - a.rho0d) * a.gd[c];  // gravity body force
                    o.u[(int64_t)c * N + n] = (float)((cl.j[c] + 0.5 * Fc) / rho);
                }
            }
        }
        cl = nl;
        cv = nv;
    }
}

// Tile and planes a block.  A block of p planes goes through p + 2 of them (the values before and
// after its own), each one load latency and its share of the CU's work: about 2 us, and 3 us for
// 1024 nodes resident on the CU, the ring's included.  A large box wants one full block a CU and
// as many planes as that leaves (256^3: 4 rows, 64 planes; with 8 planes 429 instead of 365 us a
// call); a small one wants the CUs filled by thin chunks and low tiles (p and its Laplacian, then
// rho and u, us a call with its synchronisation, against tiles of 1024 nodes and 4 planes:
// 32^3 54 + 55 -> 44 + 43, 60 x 81 x 71 62 + 58 -> 47 + 48, 128^3 82 + 78 -> 74 + 77).  Tiles whose ring has more nodes than
// the tile itself are left out (a ring node a thread).
StepGrid march_tile(const FieldArgs& a, int values, int* planes)
{
    StepGrid g;
    const int parts = (a.nx + 255) / 256;
    g.tw = (a.nx + parts - 1) / parts;  // the row in equal parts of at most 256 nodes
    g.gx = (a.nx + g.tw - 1) / g.tw;
    const int top = std::max(1, std::min(1024 / g.tw, a.ny));
    double best = -1.0;
    int th = 0;
    auto consider = [&](int h, int p) {
        const int gy = (a.ny + h - 1) / h, gz = (a.nz + p - 1) / p;
        const int64_t blocks = (int64_t)g.gx * gy * gz;
        const int threads = (g.tw * h + 63) & ~63;
        const int lds = values * 32 * (g.tw + 2) * (h + 2);
        const int fit = std::max(1, std::min(1024 / threads, 160 * 1024 / lds));
        const int64_t k = std::min<int64_t>(fit, (blocks + 255) / 256);
        const int64_t rounds = (blocks + 256 * k - 1) / (256 * k);
        const double nodes = (double)k * (threads + 2 * (g.tw + 2) + 2 * h);
        const double cost = (double)rounds * (p + 2) * (2.0 + 3.0 * nodes / 1024.0);
        if (best < 0.0 || cost < best) {
            best = cost;
            th = h;
            *planes = p;
        }
    };
    for (int h = top; h >= 1; h -= std::max(1, top / 32)) {
        if (g.tw * h < 2 * (g.tw + 2) + 2 * h) break;
        const int tiles = g.gx * ((a.ny + h - 1) / h);
        const int chunks = std::max(1, std::min(a.nz, 256 / tiles));
        consider(h, (a.nz + chunks - 1) / chunks);
        for (int p : {1, 2, 3, 4, 6, 8})
            if (p <= a.nz) consider(h, p);
    }
    if (th == 0) {  // no tile holds its ring: lanes idle
        g.tw = 32;
        th = 8;
        g.gx = (a.nx + g.tw - 1) / g.tw;
        *planes = std::min(4, a.nz);
    }
    g.th = th;
    g.gy = (a.ny + th - 1) / th;
    g.gz = (a.nz + *planes - 1) / *planes;
    return g;
}

template <int MODE>
hipError_t march3d(int storage, const void* f, const FieldOut& o, const FieldArgs& a,
                   hipStream_t st)
{
    int planes = 0;
    const StepGrid g = march_tile(a, MODE == kMixFields ? 2 : 1, &planes);
    const dim3 grid(g.gx * g.gy * g.gz), block((g.tw * g.th + 63) & ~63);
    const size_t lds = (MODE == kMixFields ? 8 : 4) * sizeof(double) * (size_t)(g.tw + 2) *
                       (size_t)(g.th + 2);
    switch (storage) {
        case SC_STORE_F32:
            hipLaunchKernelGGL((k_march3d<float, MODE>), grid, block, lds, st, (const float*)f, o,
                               a, planes, g);
            break;
        case SC_STORE_F16:
            hipLaunchKernelGGL((k_march3d<_Float16, MODE>), grid, block, lds, st,
                               (const _Float16*)f, o, a, planes, g);
            break;
        case SC_STORE_BF16:
            hipLaunchKernelGGL((k_march3d<__bf16, MODE>), grid, block, lds, st, (const __bf16*)f,
                               o, a, planes, g);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fields3d(int storage, const void* f, float* rho, float* u, const FieldArgs& a,
                           hipStream_t st)
{
    return march3d<kFields>(storage, f, FieldOut{rho, nullptr, u, nullptr, nullptr}, a, st);
}

hipError_t launch_mix_fields3d(int storage, const void* f, float* rho_l, float* rho_v, float* u,
                               const FieldArgs& a, hipStream_t st)
{
    return march3d<kMixFields>(storage, f, FieldOut{rho_l, rho_v, u, nullptr, nullptr}, a, st);
}

hipError_t launch_laplacian3d(int storage, const void* f, double* p, double* lap,
                              const FieldArgs& a, hipStream_t st)
{
    return march3d<kLaplacian>(storage, f, FieldOut{nullptr, nullptr, nullptr, p, lap}, a, st);
}

}  // namespace sc
