// shg.hip -- temperature distributions and emission of stochastically heated
// grains (Sect. 2.1.1, Appendix A: the "thermal continuous" approximation,
// cooling only into the next lower enthalpy bin, solved by forward
// substitution in double precision).
//
// For size s the photon rates per grain r_k come from a cell's absorbed
// energy in each band.  A photon k absorbed in bin i lands between the two
// bins around U_i + h nu_k, split linearly in U, so the upward rate from bin
// i to the bins >= j is
//     up[j][i] = sum_{k: target >= j} r_k + sum_{k: target in [j-1, j)} r_k f_ik.
// With the photon energies increasing along k, the first sum is a suffix sum
// sr[ks(i, j)] of r over the photons k >= ks(i, j), and the second runs over
// the photons between ks(i, j-1) and ks(i, j), f_ik = (U_i + h nu_k -
// U_{j-1}) / (U_j - U_{j-1}); ks depends only on the model and is tabulated.
// Most photons of a bin land in the bin itself or the next one (j = i + 1):
// up[i+1][i] = sum_k r_k min(U_i + h nu_k - U_i, U_{i+1} - U_i) / (U_{i+1} -
// U_i) is formed for all bins before the serial part; the later ranges hold
// a few photons at most.  No photon reaches beyond a band of bins above its
// own (the largest photon energy), so bins further below j are skipped.  The
// stationary populations follow from
//     P_j L(T_j) / (U_j - U_{j-1}) = sum_{i<j} P_i up[j][i],
// one bin after the other.  Emission per Hz: 4 pi sigma_k sum_i P_i B_nu_k(T_i)
// per grain, times the grains of the cell.
//
// Layout on the GPU.  A wave solves 16 cells, four lanes per cell; a
// workgroup of four waves goes through the sizes together, so that the
// model's tables are read from L2 about once per 64 cells.  A cell's LDS
// holds the suffix sums sr[k] of its photon rates and its populations.  With
// r_k = sr[k] - sr[k+1] every rate is a sum of suffix sums with coefficients
// >= 0 that depend on the model only:
//     up[j][i] = f_a sr[a] + sum_{a<k<b} (f_k - f_{k-1}) sr[k] + (1 - f_{b-1}) sr[b],
// a = ks(i, j-1), b = ks(i, j) (sr[b] alone when a = b).  So
//   - the first bucket, up[i+1][i] of every bin, is a matrix product (bins x
//     photons) (photons x cells) on the FP64 matrix cores;
//   - the later ranges, a few per cent of all (i, j), are a stream of
//     coefficients in the order the serial part needs them, dealt to the
//     cell's four lanes, two neighbouring photons at a time;
//   - the emission is a second matrix product (frequencies x bins) (bins x
//     cells), accumulated in registers over the sizes.
// The absorbed energies are read once and stay in registers.
//
// Measured at 32^3 cells, 25 sizes, 128 bins and 128 frequencies: 3.9 ms; the
// form before it, which evaluated the first bucket photon by photon (65000
// FP64 operations per cell and size) and the emission from LDS, 19.4 ms.
// The two products alone are 54 GFLOP, 0.75 ms at the rate of a large FP64
// matrix product; the serial part is a chain of N - 1 dependent steps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <utility>

#include "soc_kernels.h"

namespace soc {

__device__ inline double shg_planck(double nu, double T)
{
    const double h = 6.62607015e-27, k = 1.380649e-16, c = 2.99792458e10;
    const double x = h * nu / (k * T);
    const double pre = 2.0 * h * nu * nu * nu / (c * c);
    if (x > 700.0) return pre * exp(-x);
    return pre / expm1(x);
}

// Device-made model tables: rate[s][k], icool[s][i] = (U_si - U_s,i-1) /
// (4 pi sum_k sigma_sk B(nu_k, T_si) w_k), and the two products' matrices in
// the order in which a wave loads its 16 x 8 operand pieces (lane l: row l
// mod 16, reduction entries 2 (l / 16) and 2 (l / 16) + 1):
//   first[s][tile of 16 bins][8 photons][lane][2]: D_ik - D_i,k-1, D_ik =
//     min(U_i + h nu_k - U_i, U_i+1 - U_i) / (U_i+1 - U_i)
//   emit[s][tile of 16 frequencies][8 bins][lane][2]: 4 pi sigma_sk B(nu_k, T_si)
// zero beyond the model's sizes.
__global__ void shg_prep_kernel(ShgModelDev m, const double *w)
{
    const double four_pi = 12.566370614359172;
    const int S = m.S, K = m.K, N = m.N;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int nb = shg_tiles(N), nk = shg_tiles(K);   // 16-row tiles
    const int rb = shg_steps(N), rk = shg_steps(K);   // 8-entry reduction steps
    const int64_t per_emit = (int64_t)nk * rb * 128, per_first = (int64_t)nb * rk * 128;
    for (int64_t t = t0; t < S * per_emit; t += stride) {
        const int s = (int)(t / per_emit);
        const int e = (int)(t % per_emit);
        const int u = e & 1, l = (e >> 1) & 63, step = (e >> 7) % rb, tile = (e >> 7) / rb;
        const int k = 16 * tile + (l & 15), i = 8 * step + 2 * (l >> 4) + u;
        m.emit[t] = k < K && i < N ? four_pi * m.sigma[s * K + k] * shg_planck(m.nu[k], m.T[s * N + i]) : 0.0;
    }
    for (int64_t t = t0; t < S * per_first; t += stride) {
        const int s = (int)(t / per_first);
        const int e = (int)(t % per_first);
        const int u = e & 1, l = (e >> 1) & 63, step = (e >> 7) % rk, tile = (e >> 7) / rk;
        const int i = 16 * tile + (l & 15), k = 8 * step + 2 * (l >> 4) + u;
        double v = 0.0;
        if (i < N - 1 && k < K) {
            const double *U = m.U + (int64_t)s * N;
            const double dU = U[i + 1] - U[i];
            const double hi = fmin(U[i] + m.hnu[k] - U[i], dU);
            const double lo = k > 0 ? fmin(U[i] + m.hnu[k - 1] - U[i], dU) : 0.0;
            v = (hi - lo) / dU;
        }
        m.first[t] = v;
    }
    for (int64_t t = t0; t < (int64_t)S * N; t += stride) {
        const int i = (int)(t % N), s = (int)(t / N);
        double L = 0.0;
        for (int k = 0; k < K; ++k) L += four_pi * m.sigma[s * K + k] * shg_planck(m.nu[k], m.T[s * N + i]) * w[k];
        m.icool[t] = i > 0 ? (m.U[s * N + i] - m.U[s * N + i - 1]) / L : 0.0;
    }
    // rate[s][k]: photons per grain per second of size s in band k, per unit
    // of absorbed energy per H atom: the size's share of the absorption over
    // its abundance and h nu
    const int kpad = 8 * rk;
    for (int64_t t = t0; t < (int64_t)kpad; t += stride) {
        double tot = 0.0;
        if (t < K)
            for (int s = 0; s < S; ++s) tot += m.abundance[s] * m.sigma[s * K + t];
        for (int s = 0; s < S; ++s)
            m.rate[s * kpad + t] = tot > 0.0 && m.abundance[s] > 0.0
                                       ? m.abundance[s] * m.sigma[s * K + t] / tot * m.inv_hnu[t] / m.abundance[s]
                                       : 0.0;
    }
}

hipError_t launch_shg_prep(const ShgModelDev &m, const double *w, hipStream_t s)
{
    const int64_t work = (int64_t)m.S * m.N * (m.K > m.N ? m.K : m.N);
    int64_t blocks = (work + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(shg_prep_kernel, dim3((unsigned)(blocks < 1 ? 1 : blocks)), dim3(256), 0, s, m, w);
    return hipGetLastError();
}

// The coefficient stream of the later photon ranges (host).  For step j of
// size s the pairs (i, j), i <= j - 2, in order of i, each cut into pieces
// of two neighbouring photons k, k + 1; a group holds two pieces for each of
// a cell's four lanes, and a step one group at least (zero pieces fill it).
// 16 groups make a block: four planes (coefficients of the first and of the
// second pieces, LDS offsets of the first and of the second: P_i, sr[k],
// sr[k+1]) of 16 bytes for each of 64 lanes, lane 16 q + g holding lane q's
// pieces of group g.  ks(i, j), the photons of bin i whose lower target bin
// lies below j: the lower target bin of U_i + h nu_k is the last lo <= N - 2
// with U_lo <= U_i + h nu_k (at or above the top bin, all of it goes to the
// top bin), so lo >= j <=> U_j <= U_i + h nu_k for j <= N - 2, and lo never
// reaches N - 1.
void shg_build_stream(int S, int K, int N, const double *hnu, const double *U_all, ShgStream &out)
{
    out.count.assign((size_t)S * N, 0);
    out.first_block.assign(S, 0);
    out.words.clear();
    std::vector<std::vector<int>> ks(N, std::vector<int>(N, 0));
    std::vector<double> f(K + 1);
    constexpr size_t kBlock = 4 * 64 * 4;   // words
    for (int s = 0; s < S; ++s) {
        const double *U = U_all + (int64_t)s * N;
        out.first_block[s] = (int32_t)(out.words.size() / kBlock);
        const size_t base = out.words.size();
        size_t group = 0;   // of this size: the first of the step
        for (int i = 0; i < N; ++i) {
            int n = 0;
            for (int j = i; j < N; ++j) {
                if (j == N - 1) n = K;
                else while (n < K && U[i] + hnu[n] < U[j]) ++n;
                ks[j][i] = n;
            }
        }
        for (int j = 1; j < N; ++j) {
            const double dU = U[j] - U[j - 1], idu = 1.0 / dU;
            int n = 0;
            auto piece = [&](int i, int k, double c0, double c1) {
                const size_t g = group + (size_t)(n / 8);
                if (out.words.size() < base + (g / 16 + 1) * kBlock) out.words.resize(base + (g / 16 + 1) * kBlock, 0u);
                const int second = (n / 4) & 1, q = n % 4;
                uint32_t *w = &out.words[base + (g / 16) * kBlock + (size_t)second * 256 + (size_t)(16 * q + (int)(g % 16)) * 4];
                std::memcpy(w, &c0, 8);
                std::memcpy(w + 2, &c1, 8);
                w[512] = (uint32_t)(i * kShgRow);
                w[513] = (uint32_t)(shg_sr_place(k) * kShgRow);
                w[514] = (uint32_t)(shg_sr_place(k + 1) * kShgRow);
                ++n;
            };
            for (int i = 0; i <= j - 2; ++i) {
                const int a = ks[j - 1][i], b = ks[j][i];
                if (a >= K) continue;
                // coefficients of sr[a .. b] (sr[K] = 0)
                for (int k = a; k < b; ++k) f[k] = std::min(U[i] + hnu[k] - U[j - 1], dU) * idu;
                auto c = [&](int k) {
                    if (k > b || k >= K) return 0.0;
                    if (k == b) return a == b ? 1.0 : 1.0 - f[b - 1];
                    return k == a ? f[a] : f[k] - f[k - 1];
                };
                for (int k = a; k <= b && k < K; k += 2) piece(i, k, c(k), c(k + 1));
            }
            const size_t groups = std::max<size_t>(1, (size_t)(n + 7) / 8);
            out.count[(size_t)s * N + j] = (uint16_t)groups;
            group += groups;
        }
        // the kernel reads two blocks at a size's start and one block ahead
        out.words.resize(base + ((group + 15) / 16 + 2) * kBlock, 0u);
    }
}

// LDS written by some lanes of a wave and read by others: order the
// accesses within the wave.
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The value of lane I of the row.
template <int I>
__device__ inline uint32_t row_lane(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x150 + I, 0xF, 0xF, true);   // row_newbcast
}
template <int I>
__device__ inline double row_lane_f64(uint32_t lo, uint32_t hi)
{
    const long long v = (long long)((unsigned long long)hi << 32 | lo);
    const long long w = __builtin_amdgcn_update_dpp(v, v, 0x150 + I, 0xF, 0xF, true);
    return __builtin_bit_cast(double, w);
}

// f(0) && f(1) && ... with the index as a type.
template <typename F, int... I>
__device__ __forceinline__ bool all_of_16(F &f, std::integer_sequence<int, I...>)
{
    return (f(std::integral_constant<int, I>{}) && ...);
}

// A double split over the wave's four rows of 16 lanes: the value of this
// row and of the neighbouring one (Half: of the other half of the wave), in
// the lower row's order in both.
template <bool Half>
__device__ inline void row_swap(double v, double &first, double &second)
{
    const auto lo = Half ? __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false)
                         : __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto hi = Half ? __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false)
                         : __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    first = __hiloint2double(hi[0], lo[0]);
    second = __hiloint2double(hi[1], lo[1]);
}

// Sum over the four rows, in every lane.
__device__ inline double row_sum(double v)
{
    double x, y;
    row_swap<false>(v, x, y);
    row_swap<true>(x + y, x, y);
    return x + y;
}

// Sum over the later rows.
__device__ inline double later_rows(double v, int row)
{
    double x, y, a, b;
    row_swap<false>(v, x, y);       // rows 0 and 1, or 2 and 3
    row_swap<true>(x + y, a, b);    // b: rows 2 + 3
    return (row < 2 ? b : 0.0) + ((row & 1) == 0 ? y : 0.0);
}

// H atoms in a cell (n_H V); 0 outside the grid, for refined parents and
// empty cells.
__device__ inline double cell_nhv(const ShgArgs &a, int64_t cell)
{
    if (cell >= a.ncells) return 0.0;
    const uint32_t word = a.words[cell];
    const float nf = __uint_as_float(word);
    if ((int32_t)word < 0 || !(nf > 0.0f)) return 0.0;
    int lv = 0;
    while (lv + 1 < a.nlevels && cell >= a.level_offset[lv + 1]) ++lv;
    const double side = ldexp(a.root_cell_cm, -lv);
    return (double)nf * side * side * side;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kShgWaves = 4;    // waves per workgroup
constexpr int kShgCells = 16;   // cells per wave

// LDS rows (one double per cell of the wave, 128 bytes): suffix sums
// sr[0 .. K], zeros up to the padded reduction length and four more (the
// second photon of the last piece is the first of them), then the
// populations, padded likewise.  The 32 lanes that the LDS serves together
// are two lanes of each cell, which usually read the suffix sums k and
// k + 2: rows that differ in bit 1 are on different halves of the banks
// (in plain order every such pair met on one half, and the reads took as long
// as everything else).

// C[16 rows x 16 cells] of the product of one 16-row tile of `mat` with the
// operand pieces b (lane l: cell l mod 16).  Lane l holds rows 4 v + l / 16.
template <int Steps>
__device__ inline f64x4 tile_product(const double2 (&A)[Steps], const double (&b)[2 * Steps], f64x4 c)
{
#pragma unroll
    for (int t = 0; t < Steps; ++t) {
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(A[t].x, b[2 * t], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(A[t].y, b[2 * t + 1], c, 0, 0, 0);
    }
    return c;
}
template <int Steps>
__device__ inline void load_tile(const double *mat, int64_t tile, int lane, double2 (&A)[Steps])
{
    const double2 *p = (const double2 *)mat + tile * (Steps * 64) + lane;
#pragma unroll
    for (int t = 0; t < Steps; ++t) A[t] = p[t * 64];
}

// KS, NS: 8-entry reduction steps over the photons and the bins (8 or 16:
// up to 64 or 128 of them).  blockIdx.x: 64 cells; blockIdx.y: an even part
// of the sizes, whose emission goes to its own copy of the output.
template <int KS, int NS>
__global__ __launch_bounds__(64 * kShgWaves, 1) void shg_kernel(ShgArgs a)
{
    extern __shared__ double lds[];
    const ShgModelDev &m = a.model;
    const int K = m.K, N = m.N, S = m.S;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cell = lane & 15, q = lane >> 4;   // the lane's cell of the wave and its place among the cell's lanes
    constexpr int kSrRows = 8 * KS + 4, kPRows = 8 * NS + 1;
    double *const SR = lds + (size_t)wv * (kSrRows + kPRows) * kShgCells;
    double *const P = SR + kSrRows * kShgCells;
    // the size's inverse cooling rates and group counts, for the workgroup
    double *const ic = lds + (size_t)kShgWaves * (kSrRows + kPRows) * kShgCells;
    int32_t *const cnt = (int32_t *)(ic + 8 * NS);
    const int64_t c0 = ((int64_t)blockIdx.x * kShgWaves + wv) * kShgCells;
    const double nhv = cell_nhv(a, c0 + cell);
    // absorbed energy per H atom in this lane's quarter of the bands
    constexpr int KB = 2 * KS;
    const int k0 = q * KB;
    double x[KB];
    {
        const double inv = nhv > 0.0 ? 1.0 / nhv : 0.0;
#pragma unroll
        for (int i = 0; i < KB; ++i) {
            const int k = k0 + i;
            // always a load from inside the array: a branch around each would make a chain of them
            const double A = a.absorbed[(int64_t)min(k, K - 1) * a.ncells + min(c0 + cell, a.ncells - 1)];
            x[i] = k < K && nhv > 0.0 ? A * inv : 0.0;
        }
    }
    // rows that stay zero: the last four of the suffix sums (the products
    // leave zeros in the others from K and from N on)
    for (int t = lane; t < 4 * kShgCells; t += 64) SR[8 * KS * kShgCells + t] = 0.0;
    f64x4 em[KS / 2];
#pragma unroll
    for (int t = 0; t < KS / 2; ++t) em[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int s_begin = (int)((int64_t)S * blockIdx.y / gridDim.y), s_end = (int)((int64_t)S * (blockIdx.y + 1) / gridDim.y);
    for (int s = s_begin; s < s_end; ++s) {
        __syncthreads();   // the waves stay on one size, so that they share its tables in the caches
        for (int t = threadIdx.x; t < N; t += 64 * kShgWaves) {
            ic[t] = m.icool[(int64_t)s * N + t];
            cnt[t] = m.count[(int64_t)s * N + t];
        }
        // suffix sums of the photon rates: each lane sums its bands on top of the later lanes'
        if (!(m.abundance[s] > 0.0)) {   // no grains: no photons, whatever the cell absorbs (it may be no number)
#pragma unroll
            for (int i = 0; i < KB; ++i) SR[(k0 + i) * kShgCells + cell] = 0.0;
        } else {
            const double *g = m.rate + (int64_t)s * (8 * KS) + k0;   // 0 from K on
            double tot = 0.0;
#pragma unroll
            for (int i = KB - 1; i >= 0; --i) tot += x[i] * g[i];
            double acc = later_rows(tot, q);
#pragma unroll
            for (int i = KB - 1; i >= 0; --i) {
                acc += x[i] * g[i];
                SR[(k0 + shg_sr_place(i)) * kShgCells + cell] = acc;   // k0 is a multiple of 4
            }
        }
        wave_sync();
        // the first bucket: up[i+1][i] of every bin, kept in row i + 1 of the
        // populations until the population of that bin takes its place
        {
            double b[2 * KS];
#pragma unroll
            for (int t = 0; t < KS; ++t) {
                b[2 * t] = SR[shg_sr_place(8 * t + 2 * q) * kShgCells + cell];
                b[2 * t + 1] = SR[shg_sr_place(8 * t + 2 * q + 1) * kShgCells + cell];
            }
            double2 A[2][KS];
            load_tile<KS>(m.first, (int64_t)s * (NS / 2), lane, A[0]);
#pragma unroll
            for (int tile = 0; tile < NS / 2; ++tile) {
                if (tile + 1 < NS / 2) load_tile<KS>(m.first, (int64_t)s * (NS / 2) + tile + 1, lane, A[(tile + 1) & 1]);
                const f64x4 c = tile_product<KS>(A[tile & 1], b, f64x4{0.0, 0.0, 0.0, 0.0});
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    P[(16 * tile + 4 * v + q + 1) * kShgCells + cell] = c[v];
                }
            }
            if (q == 0) P[cell] = 1.0;
        }
        __syncthreads();   // the size's tables are in LDS
        // forward substitution.  The four lanes of a cell share the pieces of
        // a step; each writes the step's population, so that a lane reads
        // only what it wrote itself.  With one wave per SIMD nothing else
        // hides latencies: the stream is read a block of 16 groups ahead, a
        // group's LDS operands one group before its use (every step has a
        // group, so they belong to step j + 1 at the latest, which needs the
        // populations up to j - 1, stored before step j began), a step's other
        // inputs one step before.  A lane loads the pieces of one group of a
        // block for its row, and the row's lanes take them from each other
        // (each lane loading its own copy, 16 times the vector-memory
        // traffic: 4.4 ms instead of 3.9 ms per solve; operands two groups
        // ahead, with two groups per step: 4.5 ms).
        double tot = 1.0;
        {
            const uint4 *sp = (const uint4 *)m.stream + (int64_t)m.first_block[s] * 256 + lane;
            const char *const srl = (const char *)(SR + cell), *const pl = (const char *)(P + cell);
            struct Block { uint4 ca, cb, oa, ob; };   // coefficients and LDS offsets of the pieces a and b
            struct Operands { double pa, a0, a1, pb, b0, b1; };
            const auto load = [&] {
                const Block r = {sp[0], sp[64], sp[128], sp[192]};
                sp += 256;
                return r;
            };
            const auto fetch = [&](const Block &w, auto group) {
                constexpr int g = decltype(group)::value;
                Operands r;
                r.pa = *(const double *)(pl + row_lane<g>(w.oa.x));
                r.a0 = *(const double *)(srl + row_lane<g>(w.oa.y));
                r.a1 = *(const double *)(srl + row_lane<g>(w.oa.z));
                r.pb = *(const double *)(pl + row_lane<g>(w.ob.x));
                r.b0 = *(const double *)(srl + row_lane<g>(w.ob.y));
                r.b1 = *(const double *)(srl + row_lane<g>(w.ob.z));
                return r;
            };
            Block cur = load(), nxt = load();
            double Pj = 1.0, acc = 0.0, up1 = P[kShgCells + cell], icj = ic[1];
            int j = 1, left = __builtin_amdgcn_readfirstlane(cnt[1]), next = cnt[min(2, N - 1)];
            Operands x0 = fetch(cur, std::integral_constant<int, 0>{});
            const auto step = [&](auto group) {
                constexpr int g = decltype(group)::value;
                Operands x1 = fetch(g < 15 ? cur : nxt, std::integral_constant<int, (g + 1) % 16>{});
                acc = fma(x0.pa, fma(row_lane_f64<g>(cur.ca.x, cur.ca.y), x0.a0, row_lane_f64<g>(cur.ca.z, cur.ca.w) * x0.a1), acc);
                acc = fma(x0.pb, fma(row_lane_f64<g>(cur.cb.x, cur.cb.y), x0.b0, row_lane_f64<g>(cur.cb.z, cur.cb.w) * x0.b1), acc);
                if (--left == 0) {   // the step's population
                    acc = row_sum(acc);
                    if (__any(Pj > 1e200)) {   // keep the unnormalised populations in range
                        const double down = Pj > 1e200 ? 1e-200 : 1.0;
                        for (int i = 0; i < j; ++i) {
                            const double v = P[i * kShgCells + cell] * down;
                            wave_sync();
                            P[i * kShgCells + cell] = v;
                        }
                        Pj *= down;
                        tot *= down;
                        acc *= down;
                        x1.pa *= down;
                        x1.pb *= down;
                    }
                    Pj = fma(Pj, up1, acc) * icj;
                    P[j * kShgCells + cell] = Pj;
                    tot += Pj;
                    acc = 0.0;
                    ++j;
                    up1 = P[min(j, N - 1) * kShgCells + cell];
                    icj = ic[min(j, N - 1)];
                    left = __builtin_amdgcn_readfirstlane(next);
                    next = cnt[min(j + 1, N - 1)];
                }
                x0 = x1;
                return j < N;
            };
            while (all_of_16(step, std::make_integer_sequence<int, 16>{})) {
                cur = nxt;
                nxt = load();
            }
        }
        wave_sync();
        if (a.P) {
            for (int c = 0; c < kShgCells; ++c) {
                const double it = __shfl(nhv > 0.0 ? 1.0 / tot : 0.0, c, 64);
                if (c0 + c >= a.ncells) break;
                for (int i = lane; i < N; i += 64) a.P[((c0 + c) * S + s) * N + i] = P[i * kShgCells + c] * it;
            }
        }
        // emission: every frequency tile += (frequencies x bins) (bins x N_s P_i)
        {
            const double scale = m.abundance[s] * nhv / tot;
            double b[2 * NS];
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                b[2 * t] = P[(8 * t + 2 * q) * kShgCells + cell] * scale;
                b[2 * t + 1] = P[(8 * t + 2 * q + 1) * kShgCells + cell] * scale;
            }
            double2 A[2][NS];
            load_tile<NS>(m.emit, (int64_t)s * (KS / 2), lane, A[0]);
#pragma unroll
            for (int tile = 0; tile < KS / 2; ++tile) {
                if (tile + 1 < KS / 2) load_tile<NS>(m.emit, (int64_t)s * (KS / 2) + tile + 1, lane, A[(tile + 1) & 1]);
                em[tile] = tile_product<NS>(A[tile & 1], b, em[tile]);
            }
        }
        wave_sync();
    }
    double *out = gridDim.y > 1 ? a.part + (int64_t)blockIdx.y * K * a.ncells : a.emission;
    if (c0 + cell < a.ncells)
#pragma unroll
        for (int tile = 0; tile < KS / 2; ++tile)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = 16 * tile + 4 * v + q;
                if (k < K) out[(int64_t)k * a.ncells + c0 + cell] = em[tile][v];
            }
}

// Sum of the size parts' emissions, in order.
__global__ __launch_bounds__(256) void shg_sum_kernel(const double *part, int parts, int64_t n, double *out)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double v = 0.0;
        for (int p = 0; p < parts; ++p) v += part[(int64_t)p * n + i];
        out[i] = v;
    }
}

// Parts the sizes are cut into: a grid of fewer than 512 tiles of 64 cells
// (two per compute unit) leaves CUs idle, so its sizes are spread over more
// workgroups, each with its own emission, added up afterwards.
constexpr int64_t kShgTiles = 512;

int shg_parts(int64_t ncells, int S)
{
    const int64_t tiles = (ncells + kShgWaves * kShgCells - 1) / (kShgWaves * kShgCells);
    return (int)std::max<int64_t>(1, std::min<int64_t>(S, kShgTiles / tiles));
}

int64_t shg_part_cells(int S)
{
    return S > 1 ? kShgTiles * kShgWaves * kShgCells : 0;
}

template <int KS, int NS>
static hipError_t launch_shg_as(const ShgArgs &a, int parts, hipStream_t s)
{
    constexpr size_t lds_bytes = sizeof(double) * kShgWaves * kShgCells * (8 * (size_t)KS + 5 + 8 * NS) + 12 * 8 * (size_t)NS;
    if (lds_bytes > 65536) {   // above the default dynamic LDS limit (160 KB per CU)
        const hipError_t e = hipFuncSetAttribute((const void *)shg_kernel<KS, NS>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
    }
    const int64_t tiles = (a.ncells + kShgWaves * kShgCells - 1) / (kShgWaves * kShgCells);
    hipLaunchKernelGGL((shg_kernel<KS, NS>), dim3((unsigned)tiles, (unsigned)parts), dim3(64 * kShgWaves), lds_bytes, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || parts == 1) return e;
    const int64_t n = (int64_t)a.model.K * a.ncells;
    hipLaunchKernelGGL(shg_sum_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, s,
                       (const double *)a.part, parts, n, a.emission);
    return hipGetLastError();
}

hipError_t launch_shg(const ShgArgs &a, int parts, hipStream_t s)
{
    const bool k2 = shg_steps(a.model.K) == 16, n2 = shg_steps(a.model.N) == 16;
    if (k2 && n2) return launch_shg_as<16, 16>(a, parts, s);
    if (k2) return launch_shg_as<16, 8>(a, parts, s);
    if (n2) return launch_shg_as<8, 16>(a, parts, s);
    return launch_shg_as<8, 8>(a, parts, s);
}

}  // namespace soc
