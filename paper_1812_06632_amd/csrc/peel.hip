// peel.hip -- images of scattered light (Sect. 2.1.1: separate runs with
// forced first scattering and peel-off).
//
// Packages of the external field and the point sources are traced with the
// production emission and step code.  At every scattering the package of
// weight W at position r, moving along u, sends W Phi(u.o) exp(-tau_ext) to
// the distant observer in direction o: Phi the normalised Henyey-Greenstein
// function, tau_ext the extinction optical depth from r to the boundary
// along o (a ray march with the same step code), added to the pixel under r.
// With forced first scattering a package first measures the scattering
// optical depth tau_esc ahead of it, keeps the fraction 1 - exp(-tau_esc) of
// its weight that scatters inside the box, and draws its first free path
// from the exponential truncated at tau_esc (the same uniform that would
// otherwise give -ln u).
//
// Each lane is a small state machine: idle, transporting its package, or
// marching a ray to the boundary (the direct light of a point source, the
// escape depth of forced scattering, or a peel-off).  Every pass of the loop
// takes a step (on a regular grid four cells, and the rays to the observer in
// batches) of whichever it is doing, so long rays and long packages do not
// hold the rest of the wave; idle lanes are refilled together from a
// wave-private id pool topped up with one atomic per `chunk` ids, as in the
// Monte Carlo kernel.
#include <hip/hip_runtime.h>

#include "soc_device.h"
#include "soc_kernels.h"

namespace soc {

// Absolute position in root units on an octree: up from the leaf through the
// reverse links, halving the position and adding the octant at each level.
__device__ inline void abs_pos(const Pkg<float> &p, const McArgs &A, double &x, double &y, double &z)
{
    double fx = p.fx, fy = p.fy, fz = p.fz;
    int32_t c = p.c;
    for (int L = p.L; L > 0; --L) {
        const int o = (c - (int32_t)A.nroot) & 7;
        fx = 0.5 * (fx + (o & 1));
        fy = 0.5 * (fy + ((o >> 1) & 1));
        fz = 0.5 * (fz + ((o >> 2) & 1));
        c = A.parent[(c - A.nroot) >> 3];
    }
    x = p.cx + fx;
    y = p.cy + fy;
    z = p.cz + fz;
}

__device__ inline int64_t pixel_of(const PeelArgs &P, double x, double y, double z)
{
    int64_t i = (int64_t)floor((P.axis == 0 ? y : x) / P.psz), j = (int64_t)floor((P.axis == 2 ? y : z) / P.psz);
    i = i < 0 ? 0 : (i >= P.npx ? P.npx - 1 : i);
    j = j < 0 ? 0 : (j >= P.npy ? P.npy - 1 : j);
    return j * P.npx + i;
}

__device__ inline float hg_phase(float g, float mu)
{
    const float inv4pi = 0.0795774715459476679f;
    if (fabsf(g) < 1e-4f) return inv4pi;
    const float d = 1.0f + g * g - 2.0f * g * mu;
    return inv4pi * (1.0f - g * g) / (d * sqrtf(d));
}

enum : int { kIdle = 0, kTransport = 1, kRay = 2, kAfterDirect = 3, kWaitRay = 4 };
enum : int { kRayDirect = 0, kRayEscape = 1, kRayPeel = 2 };

// A lane's totals: summed over the wave, one set of atomics per wave that had packages.
__device__ inline void add_totals(const PeelArgs &P, unsigned long long n_pk, unsigned long long n_st, unsigned long long n_sc,
                                  unsigned long long n_ray, double e_em, double e_es)
{
    if (!__any(n_pk != 0ull)) return;
    double v[6] = {(double)n_pk, (double)n_st, (double)n_sc, (double)n_ray, e_em, e_es};
    for (int k = 0; k < 6; ++k)
        for (int off = 32; off >= 1; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
    if ((threadIdx.x & 63) == 0) {
        double *t = P.totals + 8 * (((blockIdx.x * blockDim.x + threadIdx.x) >> 6) % kStatSlots);
        for (int k = 0; k < 6; ++k) unsafeAtomicAdd(&t[k], v[k]);
    }
}

// Start a ray from the package's position along (ox, oy, oz): a probe copy
// with an infinite free path and no weight floor.
__device__ inline void ray_start(Pkg<float> &q, const Pkg<float> &p, float ox, float oy, float oz)
{
    q = p;
    q.ux = ox;
    q.uy = oy;
    q.uz = oz;
    set_inverse(q);
    q.tau = __builtin_huge_valf();
    q.W = 1.0;
    q.Wfloor = 0.0;
    q.steps = 0;
}

__global__ __launch_bounds__(256, 3) void peel_octree_kernel(McArgs A, PeelArgs P)
{
    const HG<float> hg(A.g_f);
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    unsigned long long n_pk = 0, n_st = 0, n_sc = 0, n_ray = 0;
    double e_em = 0.0, e_es = 0.0;
    // q is what the lane steps: its package, or the probe of one of the
    // package's rays while p keeps the package
    Pkg<float> p, q;
    Rng rng;
    int mode = kIdle, ray = kRayDirect, nscat = 0;
    float xi = 0.0f, rtau = 0.0f, rk = 0.0f;
    double W0 = 0.0;
    int64_t src_pix = 0;
    unsigned long long pool_next = 0, pool_end = 0;   // wave-uniform
    bool exhausted = false;                           // wave-uniform
    for (;;) {
        // refill idle lanes from the wave's id pool
        const unsigned long long idle = __ballot(mode == kIdle);
        const int nidle = __popcll(idle);
        if (!exhausted && nidle > 0) {
            const unsigned long long avail = pool_end - pool_next;
            unsigned long long grant = 0;
            if (avail < (unsigned long long)nidle) {
                const int leader = __ffsll((long long)idle) - 1;
                unsigned long long b = 0;
                if (lane == leader) b = atomicAdd(A.next_id, (unsigned long long)A.chunk);
                grant = (unsigned long long)__shfl((long long)b, leader, 64);
            }
            if (mode == kIdle) {
                const unsigned long long r = (unsigned long long)__popcll(idle & below);
                const unsigned long long id = r < avail ? pool_next + r : grant + (r - avail);
                if (id < A.n_total) {
                    uint32_t cls, pid;
                    n_pk += 1;
                    if (emit_base<float, true>(A, id, q, rng, cls, pid, W0)) {
                        e_em += W0;
                        nscat = 0;
                        xi = next_u<float>(rng, A);
                        if (P.direct && cls >= kClassPs0) {
                            const PsArg &s = A.ps[cls - kClassPs0];
                            src_pix = pixel_of(P, s.x, s.y, s.z);
                            p = q;
                            ray_start(q, p, P.ox, P.oy, P.oz);
                            ray = kRayDirect;
                            rk = A.ks_f + A.ka_f;
                            rtau = 0.0f;
                            mode = kRay;
                        } else {
                            mode = kAfterDirect;
                        }
                    }
                }
            }
            if (avail < (unsigned long long)nidle) {
                pool_next = grant + ((unsigned long long)nidle - avail);
                pool_end = grant + (unsigned long long)A.chunk;
            } else {
                pool_next += (unsigned long long)nidle;
            }
            if (pool_next >= A.n_total) exhausted = true;
        }
        // after the direct light (or at once): the escape depth, or the first free path
        if (mode == kAfterDirect) {
            if (P.forced) {
                p = q;
                ray_start(q, p, p.ux, p.uy, p.uz);
                ray = kRayEscape;
                rk = A.ks_f;
                rtau = 0.0f;
                mode = kRay;
            } else {
                q.tau = -m_log(xi);
                mode = kTransport;
            }
        }
        if (!__any(mode != kIdle)) {
            if (exhausted) break;
            continue;
        }
        if (mode == kIdle) continue;
        const float n = q.n;
        float d;
        const StepOut o = step<float, true>(q, A, A.ks_f, A.ka_f, d);
        if (mode == kRay) {
            rtau += n * rk * d;
            ++n_ray;
            if (o.event == kEvEscape || o.event == kEvRunaway) {
                q = p;   // back to the package
                if (ray == kRayDirect) {
                    unsafeAtomicAdd(&P.image[src_pix], W0 * (0.0795774715459476679 * exp(-(double)rtau)) * P.scale);
                    mode = kAfterDirect;
                } else if (ray == kRayEscape) {
                    const float qf = -expm1f(-rtau);
                    if (!(qf > 0.0f)) {
                        mode = kIdle;
                    } else {
                        q.W *= (double)qf;
                        q.tau = -log1pf(-xi * qf);
                        mode = kTransport;
                    }
                } else {   // peel-off of the scattering at q
                    const float mu = q.ux * P.ox + q.uy * P.oy + q.uz * P.oz;
                    double x, y, z;
                    abs_pos(q, A, x, y, z);
                    unsafeAtomicAdd(&P.image[pixel_of(P, x, y, z)],
                                    q.W * (double)hg_phase(A.g_f, mu) * exp(-(double)rtau) * P.scale);
                    if (P.max_scatter > 0 && ++nscat >= P.max_scatter) {
                        mode = kIdle;
                    } else {
                        scatter_new_direction<float>(q, rng, A, hg);
                        mode = kTransport;
                    }
                }
            }
        } else {
            n_st += 1;
            if (o.event == kEvEscape) {
                e_es += q.W;
                mode = kIdle;
            } else if (o.event == kEvScatter) {   // peel off towards the observer, then scatter
                n_sc += 1;
                p = q;
                ray_start(q, p, P.ox, P.oy, P.oz);
                ray = kRayPeel;
                rk = A.ks_f + A.ka_f;
                rtau = 0.0f;
                mode = kRay;
            } else if (o.event != kEvCross) {   // weight floor or step cap
                mode = kIdle;
            }
        }
    }
    add_totals(P, n_pk, n_st, n_sc, n_ray, e_em, e_es);
}

// Lanes that wait for their rays to the observer before a wave marches them
// (8 and 24 measure alike, 40 is 8% slower).
constexpr int kRayBatch = 16;

// Extinction optical depth from the package to the boundary along the
// observer's axis on a regular grid: the sum that step() gives -- the rest of
// the package's cell, then whole cells (their length is exactly 1), in FP32 in
// the order of the ray -- with the loads of 8 cells under way.  (Cells that
// are neighbours along another axis than x cost a cache line each; reading
// them from a transposed copy, 16 bytes at a time, gained nothing.)
__device__ inline float axis_ray(const Pkg<float> &q, const McArgs &A, const PeelArgs &P, float rk, unsigned long long &n_ray)
{
    // (in registers: chosen as q's members, they are chosen by address and all
    // of q lives in memory)
    int32_t cx = q.cx, cy = q.cy, cz = q.cz;
    float fx = q.fx, fy = q.fy, fz = q.fz;
    asm volatile("" : "+v"(cx), "+v"(cy), "+v"(cz), "+v"(fx), "+v"(fy), "+v"(fz));
    const bool fw = P.ox + P.oy + P.oz > 0.0f;
    const int32_t len = P.axis == 0 ? A.nx : (P.axis == 1 ? A.ny : A.nz);
    const int32_t at = P.axis == 0 ? cx : (P.axis == 1 ? cy : cz);
    const float f = P.axis == 0 ? fx : (P.axis == 1 ? fy : fz);
    const int32_t cells = (int32_t)min((int64_t)(fw ? len - at : at + 1), max(A.step_cap, (int64_t)1));
    n_ray += (unsigned long long)cells;
    float tau = q.n * rk * m_max(0.0f, fw ? 1.0f - f : f);
    const int64_t stride = (fw ? 1 : -1) * (P.axis == 0 ? (int64_t)1 : (P.axis == 1 ? (int64_t)A.nx : (int64_t)A.nx * A.ny));
    const uint32_t *const cell = A.words + (cx + A.nx * (cy + A.ny * cz));
    constexpr int kAhead = 8;
    for (int32_t k = 1; k < cells; k += kAhead) {
        float v[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) v[j] = __uint_as_float(cell[min(k + j, cells - 1) * stride]);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) tau += k + j < cells ? v[j] * rk : 0.0f;
    }
    return tau;
}

// The same on a regular grid.  A lane that wants a ray to the observer waits
// until kRayBatch lanes do (or nothing else is left to do in the wave), and
// the wave marches them together (axis_ray).  The other lanes' paths do not
// depend on the densities until the next scattering, so a pass takes each
// through kAhead cells: their lengths first, with the loads of all densities
// under way, then what happens in them, in the order and with the arithmetic
// of step(); cells behind a scattering are dropped and crossed again on
// another path (a scattering every 74 cells at 128^3).
//
// What bounds it is the latency of the loads (a cell is on another cache line
// than the last most of the time and the lines of all lanes do not fit the
// L1) and the arithmetic of a pass, at four waves per SIMD.  The 128 registers
// that these leave put 25 of the kernel's into scratch (120 bytes per lane); at
// three waves, without spills, it takes 3.38 ms against 3.45.  Measured, 128^3,
// 10^6 packages, forced first scattering, direct light of the sources (147 M
// steps of packages, 288 M of rays): 7.2 ms with the octree's kernel (every
// lane a cell per pass, three waves per SIMD, the probes of rays stepped like
// packages), of which 1.8 the atomics of the direct light on a few pixels;
// 3.4 ms here.  Cells per pass: 2 3.72, 3 3.57, 4 3.50 ms.
template <int kAhead>
__global__ __launch_bounds__(256, 4) void peel_grid_kernel(McArgs A, PeelArgs P)
{
    const HG<float> hg(A.g_f);
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    unsigned long long n_pk = 0, n_st = 0, n_sc = 0, n_ray = 0;
    double e_em = 0.0, e_es = 0.0;
    Pkg<float> q;
    Rng rng;
    int mode = kIdle, ray = kRayDirect, nscat = 0;
    float xi = 0.0f, rtau = 0.0f;
    double W0 = 0.0;
    int64_t src_pix = 0;
    // where the package stands while q goes ahead to the boundary
    int32_t bx = 0, by = 0, bz = 0;
    float gx = 0.0f, gy = 0.0f, gz = 0.0f, gn = 0.0f;
    unsigned long long pool_next = 0, pool_end = 0;   // wave-uniform
    bool exhausted = false;                           // wave-uniform
    for (;;) {
        // refill idle lanes from the wave's id pool
        const unsigned long long idle = __ballot(mode == kIdle);
        const int nidle = __popcll(idle);
        if (!exhausted && nidle > 0) {
            const unsigned long long avail = pool_end - pool_next;
            unsigned long long grant = 0;
            if (avail < (unsigned long long)nidle) {
                const int leader = __ffsll((long long)idle) - 1;
                unsigned long long b = 0;
                if (lane == leader) b = atomicAdd(A.next_id, (unsigned long long)A.chunk);
                grant = (unsigned long long)__shfl((long long)b, leader, 64);
            }
            if (mode == kIdle) {
                const unsigned long long r = (unsigned long long)__popcll(idle & below);
                const unsigned long long id = r < avail ? pool_next + r : grant + (r - avail);
                if (id < A.n_total) {
                    uint32_t cls, pid;
                    n_pk += 1;
                    if (emit_base<float, false>(A, id, q, rng, cls, pid, W0)) {
                        e_em += W0;
                        nscat = 0;
                        xi = next_u<float>(rng, A);
                        if (P.direct && cls >= kClassPs0) {
                            const PsArg &s = A.ps[cls - kClassPs0];
                            src_pix = pixel_of(P, s.x, s.y, s.z);
                            ray = kRayDirect;
                            mode = kWaitRay;
                        } else {
                            mode = kAfterDirect;
                        }
                    }
                }
            }
            if (avail < (unsigned long long)nidle) {
                pool_next = grant + ((unsigned long long)nidle - avail);
                pool_end = grant + (unsigned long long)A.chunk;
            } else {
                pool_next += (unsigned long long)nidle;
            }
            if (pool_next >= A.n_total) exhausted = true;
        }
        bool done = false;   // this lane's ray
        const int waiting = __popcll(__ballot(mode == kWaitRay));
        if (waiting >= kRayBatch || (waiting > 0 && !__any(mode == kTransport || mode == kRay || mode == kAfterDirect))) {
            if (mode == kWaitRay) {
                rtau = axis_ray(q, A, P, A.ks_f + A.ka_f, n_ray);
                done = true;
            }
        }
        // after the direct light (or at once): the escape depth, or the first free path
        if (mode == kAfterDirect) {
            if (P.forced) {
                bx = q.cx, by = q.cy, bz = q.cz;
                gx = q.fx, gy = q.fy, gz = q.fz, gn = q.n;
                ray = kRayEscape;
                rtau = 0.0f;
                mode = kRay;
            } else {
                q.tau = -m_log(xi);
                mode = kTransport;
            }
        }
        if (!__any(mode != kIdle)) {
            if (exhausted) break;
            continue;
        }
        if (mode == kTransport || mode == kRay) {
            int32_t cx[kAhead + 1], cy[kAhead + 1], cz[kAhead + 1], c = 0;
            float fx[kAhead + 1], fy[kAhead + 1], fz[kAhead + 1], n[kAhead + 1], d[kAhead];
            bool leaves[kAhead], inside = true;
            cx[0] = q.cx, cy[0] = q.cy, cz[0] = q.cz;
            fx[0] = q.fx, fy[0] = q.fy, fz[0] = q.fz, n[0] = q.n;
            const bool px = q.ux > 0.0f, py = q.uy > 0.0f, pz = q.uz > 0.0f;
#pragma unroll
            for (int j = 0; j < kAhead; ++j) {
                const float dx = (q.tx - fx[j]) * q.ix, dy = (q.ty - fy[j]) * q.iy, dz = (q.tz - fz[j]) * q.iz;
                const bool ax = (dx <= dy) & (dx <= dz), ay = !ax & (dy <= dz), az = !ax & !ay;
                d[j] = m_max(0.0f, ax ? dx : (ay ? dy : dz));
                fx[j + 1] = ax ? (px ? 0.0f : 1.0f) : m_clamp01(fx[j] + d[j] * q.ux);
                fy[j + 1] = ay ? (py ? 0.0f : 1.0f) : m_clamp01(fy[j] + d[j] * q.uy);
                fz[j + 1] = az ? (pz ? 0.0f : 1.0f) : m_clamp01(fz[j] + d[j] * q.uz);
                cx[j + 1] = cx[j] + (ax ? (px ? 1 : -1) : 0);
                cy[j + 1] = cy[j] + (ay ? (py ? 1 : -1) : 0);
                cz[j + 1] = cz[j] + (az ? (pz ? 1 : -1) : 0);
                inside &= ((uint32_t)cx[j + 1] < (uint32_t)A.nx) & ((uint32_t)cy[j + 1] < (uint32_t)A.ny) &
                          ((uint32_t)cz[j + 1] < (uint32_t)A.nz);
                leaves[j] = !inside;
                c = inside ? cx[j + 1] + A.nx * (cy[j + 1] + A.ny * cz[j + 1]) : c;   // outside: a load that is not used
                n[j + 1] = __uint_as_float(A.words[c]);
            }
            int at = kAhead;   // the cell in which something happens
            int ev = kEvCross;
            float ds = 0.0f;
            if (mode == kRay) {
#pragma unroll
                for (int j = 0; j < kAhead; ++j) {
                    if (done) continue;
                    rtau += n[j] * A.ks_f * d[j];
                    ++n_ray;
                    q.steps += 1;
                    done = leaves[j] || (int64_t)q.steps >= A.step_cap;
                }
            } else {
#pragma unroll
                for (int j = 0; j < kAhead; ++j) {
                    if (ev != kEvCross) continue;
                    const float ks = n[j] * A.ks_f, ka = n[j] * A.ka_f;
                    const float tcell = ks * d[j];
                    ds = d[j];
                    if (ks > 0.0f && tcell >= q.tau) {
                        ds = m_min(q.tau * m_rcp(ks), d[j]);
                        ev = kEvScatter;
                    } else {
                        q.tau -= tcell;
                        if (leaves[j]) ev = kEvEscape;
                    }
                    q.W -= q.W * (double)one_minus_exp_neg(ka * ds);
                    q.steps += 1;
                    n_st += 1;
                    if (ev != kEvEscape) {
                        if (fabs(q.W) < q.Wfloor) ev = kEvFloor;
                        else if ((int64_t)q.steps >= A.step_cap) ev = kEvRunaway;
                    }
                    if (ev != kEvCross) at = j;
                }
            }
#pragma unroll
            for (int j = 0; j <= kAhead; ++j)
                if (at == j) {
                    q.cx = cx[j], q.cy = cy[j], q.cz = cz[j];
                    q.fx = fx[j], q.fy = fy[j], q.fz = fz[j], q.n = n[j];
                }
            if (done) {   // back to the package
                q.cx = bx, q.cy = by, q.cz = bz;
                q.fx = gx, q.fy = gy, q.fz = gz, q.n = gn;
                q.steps = 0;
            } else if (ev == kEvScatter) {   // peel off towards the observer, then scatter
                q.fx = m_clamp01(q.fx + ds * q.ux);
                q.fy = m_clamp01(q.fy + ds * q.uy);
                q.fz = m_clamp01(q.fz + ds * q.uz);
                n_sc += 1;
                ray = kRayPeel;
                mode = kWaitRay;
            } else if (ev != kEvCross) {   // out of the box, weight floor or step cap
                if (ev == kEvEscape) e_es += q.W;
                mode = kIdle;
            }
        }
        bool direct = false;
        double light = 0.0;
        if (done) {
            if (ray == kRayDirect) {
                light = W0 * (0.0795774715459476679 * exp(-(double)rtau)) * P.scale;
                direct = true;
                mode = kAfterDirect;
            } else if (ray == kRayEscape) {
                const float qf = -expm1f(-rtau);
                if (!(qf > 0.0f)) {
                    mode = kIdle;
                } else {
                    q.W *= (double)qf;
                    q.tau = -log1pf(-xi * qf);
                    mode = kTransport;
                }
            } else {   // peel-off of the scattering at q
                const float mu = q.ux * P.ox + q.uy * P.oy + q.uz * P.oz;
                unsafeAtomicAdd(&P.image[pixel_of(P, (double)q.cx + (double)q.fx, (double)q.cy + (double)q.fy, (double)q.cz + (double)q.fz)],
                                q.W * (double)hg_phase(A.g_f, mu) * exp(-(double)rtau) * P.scale);
                if (P.max_scatter > 0 && ++nscat >= P.max_scatter) {
                    mode = kIdle;
                } else {
                    scatter_new_direction<float>(q, rng, A, hg);
                    mode = kTransport;
                }
            }
        }
        // a source's direct light goes to one pixel: one atomic per wave and
        // source (half a million atomics on a pixel took 2 ms)
        for (unsigned long long m = __ballot(direct); m;) {
            const int64_t pix = __shfl(src_pix, __ffsll((long long)m) - 1, 64);
            const bool mine = direct && src_pix == pix;
            double sum = mine ? light : 0.0;
            for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
            if (lane == 0) unsafeAtomicAdd(&P.image[pix], sum);
            m &= ~__ballot(mine);
        }
    }
    add_totals(P, n_pk, n_st, n_sc, n_ray, e_em, e_es);
}

hipError_t launch_peel(const McArgs &a, const PeelArgs &p, int blocks, hipStream_t s)
{
    if (a.nlevels > 1) hipLaunchKernelGGL(peel_octree_kernel, dim3(blocks), dim3(256), 0, s, a, p);
    else hipLaunchKernelGGL(peel_grid_kernel<4>, dim3(blocks), dim3(256), 0, s, a, p);
    return hipGetLastError();
}

}  // namespace soc
