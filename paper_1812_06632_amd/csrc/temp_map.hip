// temp_map.hip -- equilibrium dust temperature and emission maps
// (Juvela 2019, Sect. 2.1.1: separate kernels solve the dust temperature
// from the frequency-integrated absorbed energy and make surface-brightness
// maps from that solution).
//
// Temperature: Gamma(T) = 4 pi sum_k w_k sigma_abs,k B_nu_k(T) is tabulated
// once on a log-T grid; each cell inverts ln Gamma -> ln T by a search in
// the table and linear interpolation in the log-log plane.  The pass streams
// over the cells (A: 8 B, word: 4 B, T_old: 4 B, T_new: 4 B).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "soc_kernels.h"

namespace soc {

__device__ inline double planck_b(double nu, double T)
{
    const double h = 6.62607015e-27, k = 1.380649e-16, c = 2.99792458e10;
    if (!(T > 0.0)) return 0.0;
    const double x = h * nu / (k * T);
    const double pre = 2.0 * h * nu * nu * nu / (c * c);
    if (x > 700.0) return pre * exp(-x);
    return pre / expm1(x);
}

__global__ void temp_table_kernel(const double *nu, const double *w, const double *sabs, int32_t K, double lnTf,
                                  double dlnT, int32_t nT, double *lnG)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nT) return;
    const double T = exp(lnTf + dlnT * j);
    double s = 0.0;
    for (int k = 0; k < K; ++k) s += w[k] * sabs[k] * planck_b(nu[k], T);
    lnG[j] = log(12.566370614359172 * s);
}

// Search starts: for each of kTempStarts equal steps of ln Gamma the last
// entry safely below the step's lower edge (the margins cover the rounding
// of the edge and of the solve's step number), at most nT - 2.
__global__ void temp_starts_kernel(const double *lnG, int32_t nT, uint16_t *start)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= kTempStarts) return;
    const double G0 = lnG[0], Gn = lnG[nT - 1];
    const double edge = G0 + (b - 1e-9) * ((Gn - G0) / kTempStarts) - 1e-15 * (fabs(G0) + fabs(Gn));
    int lo = 0, hi = nT - 1;   // lnG[lo] <= edge (or lo == 0), lnG[hi] > edge
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (lnG[mid] <= edge) lo = mid; else hi = mid;
    }
    start[b] = (uint16_t)lo;
}

hipError_t launch_temp_table(const double *nu, const double *w, const double *sabs, int32_t K, double lnTf,
                             double dlnT, int32_t nT, double *lnG, uint16_t *start, hipStream_t s)
{
    hipLaunchKernelGGL(temp_table_kernel, dim3((nT + 255) / 256), dim3(256), 0, s, nu, w, sabs, K, lnTf, dlnT, nT, lnG);
    hipLaunchKernelGGL(temp_starts_kernel, dim3(kTempStarts / 256), dim3(256), 0, s, (const double *)lnG, nT, start);
    return hipGetLastError();
}

__device__ inline int level_index(int64_t c, const int64_t *lo, int32_t nlevels)
{
    int L = 0;
    while (L + 1 < nlevels && c >= lo[L + 1]) ++L;
    return L;
}

// 512-lane workgroups, two per compute unit: 16 waves per CU hide the
// chains of FP64 divisions, logarithm and exponential of a cell (256 lanes,
// 8 waves per CU: 56 us for the update pass at 128^3).
constexpr int kTempThreads = 512;

// Histogram key of a temperature.  The bit pattern of a float >= 0 grows
// with its value, so a coarse bin is a range of 2^sh consecutive floats
// counted from bit pattern b0 (2^sh-aligned, so that a bin never spans two
// exponents) and the fine bins divide it evenly: no logarithm is taken.
// Values outside the table's range fall into the end bins.
__device__ inline int coarse_bin(float T, uint32_t b0, int sh)
{
    const uint32_t u = __float_as_uint(fmaxf(T, 0.0f));
    const uint32_t b = u > b0 ? (u - b0) >> sh : 0u;
    return b >= (uint32_t)kHistBins ? kHistBins - 1 : (int)b;
}
__device__ inline int fine_bin(float T, int tb, uint32_t b0, int sh)
{
    const uint32_t u = __float_as_uint(fmaxf(T, 0.0f)), lo = b0 + ((uint32_t)tb << sh);
    const uint32_t b = u > lo ? (u - lo) >> (sh - kFineBits) : 0u;
    return b >= (uint32_t)kFineBins ? kFineBins - 1 : (int)b;
}

// Sum over the wave, in every lane; fixed order.
__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Temperature of every leaf (given: T_new already holds the temperatures
// and only the statistics are taken).  With statistics requested, each
// workgroup writes its partial sums (count, sum T, sum |dT|/T_old, count with
// T_old > 0, clamped) to its own row and adds its LDS histogram of the
// temperatures to the total, whose integer adds give the same result in any
// order.
//
// Bound: FP64 arithmetic (about 250 vector instructions per cell: three
// divisions, a logarithm, an exponential) next to 20 bytes per cell.  The
// table's interval is found through a start index per equal step of
// ln Gamma (one or two table reads instead of a 12-step binary search).
// Staged: the table and its start indices are copied to LDS, worth it once
// a lane has several cells; a small grid reads them through L2.
// A solve with statistics of 128^3 cells: 66 us (with the passes below and
// the wait for the result; 421 us with logarithmic bins, one histogram row
// per workgroup and serial sums over the rows).
template <bool Staged>
__global__ __launch_bounds__(kTempThreads) void temp_update_kernel(TempArgs a)
{
    __shared__ double sh_lnG[Staged ? kTempMaxT : 1];
    __shared__ uint16_t sh_start[Staged ? kTempStarts : 1];
    __shared__ unsigned int sh_hist[kHistBins];
    __shared__ double sh_red[kTempThreads / 64][5];
    const bool want = a.part != nullptr;
    if (Staged && !a.given) {
        for (int j = threadIdx.x; j < a.nT; j += kTempThreads) sh_lnG[j] = a.lnG[j];
        for (int j = threadIdx.x; j < kTempStarts; j += kTempThreads) sh_start[j] = a.start[j];
    }
    if (want)
        for (int j = threadIdx.x; j < kHistBins; j += kTempThreads) sh_hist[j] = 0u;
    __syncthreads();
    double cnt = 0.0, sumT = 0.0, sumrel = 0.0, nrel = 0.0, ncl = 0.0;
    for (int64_t c = (int64_t)blockIdx.x * kTempThreads + threadIdx.x; c < a.ncells; c += (int64_t)gridDim.x * kTempThreads) {
        const uint32_t w = a.words[c];
        const float nf = __uint_as_float(w);
        float Tout = 0.0f;
        if ((int32_t)w >= 0 && nf > 0.0f) {
            double T;
            bool clamped = false;
            if (a.given) {
                T = (double)a.T_new[c];
            } else {
                const int L = level_index(c, a.level_offset, a.nlevels);
                const double s = ldexp(a.root_cell_cm, -L);
                double y = a.absorbed[c] / ((double)nf * (s * s * s));
                if (a.ali_self) {
                    // diagonal ALI: the cell re-absorbs the fraction self/emitted of its own
                    // emission, so its emission is the absorption from elsewhere over the
                    // escape probability (kept >= 1e-6)
                    const double e = a.ali_emit[c];
                    const double esc = e > 0.0 ? fmax(1.0 - a.ali_self[c] / e, 1e-6) : 1.0;
                    y /= esc;
                }
                if (!(y > 0.0)) {
                    T = a.T_floor;
                    clamped = true;
                } else {
                    const double ly = log(y);
                    if (!(ly > a.G0)) {
                        T = a.T_floor;
                        clamped = true;
                    } else if (ly >= a.Gn) {
                        T = a.T_max;
                        clamped = true;
                    } else {
                        // lnG[lo] <= ly < lnG[lo + 1]; the start index is at or below lo
                        const int b = min((int)((ly - a.G0) * a.start_scale), kTempStarts - 1);
                        int lo = Staged ? sh_start[b] : a.start[b];
                        double g0 = Staged ? sh_lnG[lo] : a.lnG[lo], g1 = Staged ? sh_lnG[lo + 1] : a.lnG[lo + 1];
                        while (g1 <= ly) {
                            ++lo;
                            g0 = g1;
                            g1 = Staged ? sh_lnG[lo + 1] : a.lnG[lo + 1];
                        }
                        const double t = (ly - g0) / (g1 - g0);
                        T = exp(a.lnTf + a.dlnT * ((double)lo + t));
                    }
                }
            }
            Tout = (float)T;
            if (want) {
                const double Tf = (double)Tout;
                cnt += 1.0;
                sumT += Tf;
                ncl += clamped ? 1.0 : 0.0;
                if (a.T_old) {
                    const float To = a.T_old[c];
                    if (To > 0.0f) {
                        sumrel += fabs(Tf - (double)To) / (double)To;
                        nrel += 1.0;
                    }
                }
                atomicAdd(&sh_hist[coarse_bin(Tout, a.b0, a.sh)], 1u);
            }
        }
        if (!a.given) a.T_new[c] = Tout;
    }
    if (!want) return;
    cnt = wave_sum(cnt);
    sumT = wave_sum(sumT);
    sumrel = wave_sum(sumrel);
    nrel = wave_sum(nrel);
    ncl = wave_sum(ncl);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh_red[wv][0] = cnt;
        sh_red[wv][1] = sumT;
        sh_red[wv][2] = sumrel;
        sh_red[wv][3] = nrel;
        sh_red[wv][4] = ncl;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        double v = 0.0;
        for (int k = 0; k < kTempThreads / 64; ++k) v += sh_red[k][threadIdx.x];
        a.part[(int64_t)blockIdx.x * 8 + threadIdx.x] = v;
    }
    for (int j = threadIdx.x; j < kHistBins; j += kTempThreads)
        if (sh_hist[j]) atomicAdd(&a.hist_total[j], sh_hist[j]);
}

hipError_t launch_temp_update(const TempArgs &a, hipStream_t s)
{
    if (a.given || a.ncells < 4ll * kTempThreads * a.blocks)
        hipLaunchKernelGGL(temp_update_kernel<false>, dim3((unsigned)a.blocks), dim3(kTempThreads), 0, s, a);
    else
        hipLaunchKernelGGL(temp_update_kernel<true>, dim3((unsigned)a.blocks), dim3(kTempThreads), 0, s, a);
    return hipGetLastError();
}

int32_t temp_blocks(int64_t ncells)
{
    const int64_t b = (ncells + kTempThreads - 1) / kTempThreads;
    return (int32_t)(b < 1 ? 1 : (b < kTempBlocks ? b : kTempBlocks));
}

// One workgroup's exclusive scan of one value per lane over 1024 lanes:
// within each wave by shuffles, then over the 16 wave totals.  (Not the
// inclusive scan less the lane's own value, which is no number where that is
// infinite.)
constexpr int kFinThreads = 1024;

__device__ inline double block_scan(double v, double *sh)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    if (lane == 63) sh[wv] = v;
    __syncthreads();
    double base = 0.0;
    for (int k = 0; k < wv; ++k) base += sh[k];
    __syncthreads();
    const double before = __shfl_up(v, 1, 64);
    return base + (lane > 0 ? before : 0.0);
}

// Sum over the workgroups' rows of columns col .. col + n - 1 of `part`
// (at most 512 rows): result in sh_p of every lane, fixed order.
template <int N>
__device__ inline void sum_parts(const TempArgs &a, int col, double (*sh)[8], double *sh_p)
{
    const int t = threadIdx.x, wv = t >> 6;
    double v[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        v[q] = t < a.blocks ? a.part[(int64_t)t * 8 + col + q] : 0.0;
        v[q] = wave_sum(v[q]);
        if ((t & 63) == 0) sh[wv][q] = v[q];
    }
    __syncthreads();
    if (t < N) {
        double s = 0.0;
        for (int k = 0; k < kFinThreads / 64; ++k) s += sh[k][t];
        sh_p[t] = s;
    }
    __syncthreads();
}

// Reduce the per-workgroup partial sums, then locate the coarse bin holding
// the k-th hottest leaf (k = ceil(0.05 n)).  One workgroup; the sums over
// the rows and the scan over the bins are a few shuffles each (serial loops
// over 512 rows took 79 us here and 105 us in the finish).
// meta: [0] count [1] sum T [2] sum rel [3] n rel [4] clamped
//       [5] threshold bin [6] cells still needed from that bin [7] k
constexpr int kFinPer = kHistBins / kFinThreads;

__global__ __launch_bounds__(kFinThreads) void temp_stats_reduce_kernel(TempArgs a)
{
    __shared__ double sh[kFinThreads / 64][8];
    __shared__ double sh_p[8];
    __shared__ double sh_s[kFinThreads / 64];
    const int t = threadIdx.x;
    sum_parts<5>(a, 0, sh, sh_p);
    // lane t covers bins [hi - per, hi), counted from the top
    const int hi = kHistBins - t * kFinPer;
    double loc[kFinPer];
    double n = 0.0;
    for (int q = 0; q < kFinPer; ++q) {
        loc[q] = (double)a.hist_total[hi - 1 - q];
        a.hist_total[hi - 1 - q] = 0u;   // left zero for the next call
        n += loc[q];
    }
    const double before = block_scan(n, sh_s);
    const double count = sh_p[0];
    const double k = ceil(0.05 * count);
    if (count > 0.0 && before < k && before + n >= k) {
        double cn = before;
        for (int q = 0; q < kFinPer; ++q) {
            if (cn + loc[q] >= k) {
                a.meta[5] = (double)(hi - 1 - q);
                a.meta[6] = k - cn;
                break;
            }
            cn += loc[q];
        }
    }
    if (t < 5) a.meta[t] = sh_p[t];
    if (t == 0) {
        a.meta[7] = k;
        if (!(count > 0.0)) {
            a.meta[5] = (double)kHistBins;
            a.meta[6] = 0.0;
        }
    }
}

// Second pass over the temperatures: exact sum of T above the threshold
// bin (per-workgroup partials) and a fine histogram (counts and sums) of
// the cells inside it, which are few.
__global__ __launch_bounds__(kTempThreads) void temp_stats_refine_kernel(TempArgs a)
{
    __shared__ double sh[kTempThreads / 64];
    const int tb = (int)a.meta[5];
    double above = 0.0;
    for (int64_t c = (int64_t)blockIdx.x * kTempThreads + threadIdx.x; c < a.ncells; c += (int64_t)gridDim.x * kTempThreads) {
        const uint32_t w = a.words[c];
        const float T = a.T_new[c];
        if ((int32_t)w < 0 || !(__uint_as_float(w) > 0.0f)) continue;
        const int b = coarse_bin(T, a.b0, a.sh);
        if (b > tb) {
            above += (double)T;
        } else if (b == tb) {
            const int f = fine_bin(T, tb, a.b0, a.sh);
            atomicAdd(&a.fine_n[f], 1u);
            unsafeAtomicAdd(&a.fine_T[f], (double)T);
        }
    }
    above = wave_sum(above);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = above;
    __syncthreads();
    if (threadIdx.x == 0) {
        double v = 0.0;
        for (int k = 0; k < kTempThreads / 64; ++k) v += sh[k];
        a.part[(int64_t)blockIdx.x * 8 + 5] = v;
    }
}

// Final statistics: mean T, hottest-5% mean (cells above the threshold bin
// plus the hottest cells inside it, resolved on the fine histogram, whose
// bins hold a few neighbouring floats), mean relative change, clamps.
// `out` is pinned host memory: the result needs no copy.
constexpr int kFinePer = kFineBins / kFinThreads;

__global__ __launch_bounds__(kFinThreads) void temp_stats_finish_kernel(TempArgs a, double *out)
{
    __shared__ double sh[kFinThreads / 64][8];
    __shared__ double sh_p[8];
    __shared__ double sh_s[kFinThreads / 64];
    const int t = threadIdx.x;
    sum_parts<1>(a, 5, sh, sh_p);
    const double above = sh_p[0];
    const int hi = kFineBins - t * kFinePer;
    double bn[kFinePer], bT[kFinePer];
    double n = 0.0, sT = 0.0;
    for (int q = 0; q < kFinePer; ++q) {
        const int b = hi - 1 - q;
        bn[q] = (double)a.fine_n[b];
        bT[q] = a.fine_T[b];
        a.fine_n[b] = 0u;   // left zero for the next call
        a.fine_T[b] = 0.0;
        n += bn[q];
        sT += bT[q];
    }
    const double before_n = block_scan(n, sh_s), before_T = block_scan(sT, sh_s);
    const double count = a.meta[0];
    const double need = a.meta[6];
    const double k = a.meta[7];
    if (count > 0.0 && need > 0.0 && before_n < need && before_n + n >= need) {
        double cn = before_n, cT = before_T;
        for (int q = 0; q < kFinePer; ++q) {
            if (cn + bn[q] >= need) {
                cT += (need - cn) * (bT[q] / bn[q]);
                break;
            }
            cn += bn[q];
            cT += bT[q];
        }
        out[1] = (above + cT) / k;
    }
    if (t == 0) {
        out[0] = count > 0.0 ? a.meta[1] / count : 0.0;
        out[2] = a.meta[3] > 0.0 ? a.meta[2] / a.meta[3] : __builtin_nan("");
        out[3] = a.meta[4];
        if (!(count > 0.0)) out[1] = 0.0;
        else if (!(need > 0.0)) out[1] = above / k;
    }
}

hipError_t launch_temp_stats(const TempArgs &a, double *out4, hipStream_t s)
{
    hipLaunchKernelGGL(temp_stats_reduce_kernel, dim3(1), dim3(kFinThreads), 0, s, a);
    hipLaunchKernelGGL(temp_stats_refine_kernel, dim3((unsigned)a.blocks), dim3(kTempThreads), 0, s, a);
    hipLaunchKernelGGL(temp_stats_finish_kernel, dim3(1), dim3(kFinThreads), 0, s, a, out4);
    return hipGetLastError();
}

// ------------------------------------------------------------------ map
// Pixel = finest cell.  The ray runs along the axis from the observer side;
// each leaf on it adds S (1 - e^{-dtau}) e^{-tau}, S = (sigma_abs /
// sigma_ext) B_nu(T), accumulated in FP64.
__device__ inline int64_t leaf_lookup(const uint32_t *words, int32_t nx, int32_t ny, double px, double py, double pz,
                                      double &lox, double &loy, double &loz, double &size)
{
    const int64_t ix = (int64_t)floor(px), iy = (int64_t)floor(py), iz = (int64_t)floor(pz);
    int64_t c = ix + (int64_t)nx * (iy + (int64_t)ny * iz);
    lox = (double)ix; loy = (double)iy; loz = (double)iz; size = 1.0;
    int32_t w = (int32_t)words[c];
    while (w < 0) {
        const int64_t first = -(int64_t)w;
        size *= 0.5;
        const int ox = px >= lox + size, oy = py >= loy + size, oz = pz >= loz + size;
        lox += ox * size; loy += oy * size; loz += oz * size;
        c = first + ox + 2 * oy + 4 * oz;
        w = (int32_t)words[c];
    }
    return c;
}

// A ray is cut into blockDim.y parts of whole root cells (in which its
// leaves nest): lane (x, y) integrates part y of pixel x, with its emission
// I and its transmission E, and the parts are joined from the observer's
// side, I_0 + E_0 (I_1 + E_1 (...)).  A cell's factor of E
// is 1 - (1 - e^{-dtau}) only while that keeps its digits: behind an opaque
// cell it has none left, and the cell's own light may be weaker still.  Bound: the latency of a cell's chain
// (dependent loads of the leaf's words, two FP64 exponentials); one lane per
// ray left 256 waves for a 128^2 image: 61 us for 32^3 root cells with three
// levels, 15 us in parts.
constexpr int kMapPixels = 64;
constexpr int kMapParts = 16;

__global__ __launch_bounds__(kMapPixels * kMapParts) void map_kernel(MapArgs a)
{
    __shared__ double sh_I[kMapParts][kMapPixels], sh_E[kMapParts][kMapPixels];
    const int i = blockIdx.x * kMapPixels + threadIdx.x;
    const int j = blockIdx.y;
    const int part = threadIdx.y, parts = blockDim.y;
    const int ax = a.axis;
    const int bx = ax == 0 ? 1 : 0, cx = ax == 2 ? 1 : 2;
    const int32_t N[3] = {a.nx, a.ny, a.nz};
    const double psz = ldexp(1.0, -(a.nlevels - 1));
    double I = 0.0, E = 1.0;
    if (i < a.npx && a.sigma_ext > 0.0) {
        double p[3];
        p[bx] = (i + 0.5) * psz;
        p[cx] = (j + 0.5) * psz;
        // root cells [n0, n1) of the ray, counted from the observer
        const int n0 = (int)((int64_t)N[ax] * part / parts), n1 = (int)((int64_t)N[ax] * (part + 1) / parts);
        double x = a.neg ? n0 : N[ax] - n0;
        const double end = a.neg ? n1 : N[ax] - n1;
        const double half = 0.5 * ldexp(1.0, -(a.nlevels + 1));   // quarter of the finest cell
        while (a.neg ? (x < end) : (x > end)) {
            p[ax] = a.neg ? x + half : x - half;
            double lo[3], size;
            const int64_t c = leaf_lookup(a.words, a.nx, a.ny, p[0], p[1], p[2], lo[0], lo[1], lo[2], size);
            const double xn = a.neg ? lo[ax] + size : lo[ax];
            const double ds = fabs(xn - x);
            const float nf = __uint_as_float(a.words[c]);
            if (nf > 0.0f) {
                const double dt = a.sigma_ext * (double)nf * ds * a.root_cell_cm;
                const double S = (a.sigma_abs / a.sigma_ext) * planck_b(a.nu, (double)a.T[c]);
                const double loss = -expm1(-dt);
                I += S * loss * E;
                E *= dt < 0.5 ? 1.0 - loss : exp(-dt);
            }
            x = xn;
        }
    }
    sh_I[part][threadIdx.x] = I;
    sh_E[part][threadIdx.x] = E;
    __syncthreads();
    if (part != 0 || i >= a.npx) return;
    double sum = 0.0;
    for (int k = parts - 1; k >= 0; --k) sum = sh_I[k][threadIdx.x] + sh_E[k][threadIdx.x] * sum;
    a.image[(int64_t)j * a.npx + i] = (float)sum;
}

hipError_t launch_map(const MapArgs &a, hipStream_t s)
{
    // parts: about 16 waves per compute unit in all, at most one per root cell
    const int32_t n = a.axis == 0 ? a.nx : (a.axis == 1 ? a.ny : a.nz);
    const int64_t rows = (int64_t)((a.npx + kMapPixels - 1) / kMapPixels) * a.npy;
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(kMapParts, n), 4096 / rows));
    hipLaunchKernelGGL(map_kernel, dim3((a.npx + kMapPixels - 1) / kMapPixels, a.npy), dim3(kMapPixels, (unsigned)parts), 0, s, a);
    return hipGetLastError();
}

}  // namespace soc
