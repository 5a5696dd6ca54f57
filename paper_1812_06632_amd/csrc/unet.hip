// unet.hip -- BF16 MFMA kernels and runtime of the 3-D U-Net surrogate.
//
// Every convolution of the network, forward and backward-data alike, is one
// implicit GEMM: rows are the positions of a "row grid", columns the output
// channels, and the reduction runs over (tap, input channel) pairs.  A
// layer kind only changes how a row maps to input and output positions:
//   3^3 convolution        rows = grid,        input = row + tap - 1,   output = row
//   stride-2 2^3 (down)    rows = coarse grid, input = 2 row + tap,     output = row
//   transposed 2^3 (up)    rows = coarse grid, input = row,             output = 2 row + phase
// (a transposed convolution is eight independent phase GEMMs).  The
// backward-data pass of each kind is again one of these forms with the
// weights re-laid out (flipped taps for the 3^3 convolution, phases and taps
// exchanged between the up and down convolutions).
//
// Each wave computes 32-row x 32-column tiles with
// v_mfma_f32_32x32x16_bf16 (8 BF16 of A and B per lane, 16 FP32 results
// per lane); operands are 16-byte vectors per lane: 8 consecutive input
// channels of one position of a channels-last tensor (A) and 8 consecutive
// reduction entries of one output channel (B, the weights laid out in
// operand order).  The epilogue adds the bias, applies the leaky
// ReLU, or -- in backward-data passes -- multiplies by the leaky ReLU
// derivative taken from the sign of the stored activation and adds a
// second gradient (the skip connection), then rounds to BF16.
//
// Weight gradients contract over positions: each workgroup reduces a chunk
// of positions for a 32 x 32 (input, output channel) tile and one tap (all 27
// of a 3^3 layer), transposing the channels-last tiles through LDS, and writes
// a partial sum;
// a second kernel adds the partials in a fixed order, so training is
// bit-reproducible.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <type_traits>

#include "unet.h"

namespace soc {
namespace unet {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kLeak = 0.1f;

__device__ __host__ inline uint16_t f2bf(float f)
{
    uint32_t u;
    memcpy(&u, &f, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;   // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);                      // round to nearest, ties to even
    return (uint16_t)(u >> 16);
}

__device__ __host__ inline float bf2f(uint16_t h)
{
    const uint32_t u = (uint32_t)h << 16;
    float f;
    memcpy(&f, &u, 4);
    return f;
}

__device__ inline bf16x8_t ld8(const uint16_t *p)
{
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4 *>(p));
}

__device__ inline bf16x8_t zero8()
{
    return __builtin_bit_cast(bf16x8_t, u32x4{0u, 0u, 0u, 0u});
}

// Workgroup barrier for LDS alone: __syncthreads also waits for every load
// from memory, among them those made for the next round.
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ------------------------------------------------------------------ conv
struct ConvArgs {
    const uint16_t *x;
    int32_t x_cs, x_co, cin;        // input view; cin channels per tap (multiple of 16)
    int32_t iz, iy, ix;             // input grid of one sample
    int32_t mz, my, mx, batch;      // row grid of one sample, samples
    int32_t k, s_in, pad;           // taps per axis, input stride, padding
    int32_t nph, s_out;             // output phases (1 or 8), output stride
    int32_t oz, oy, ox;             // output grid of one sample
    const uint16_t *w;              // weight operands, see weight_operand
    int32_t npad;
    const float *bias;              // NULL: none
    int32_t cout;                   // columns stored (n < cout)
    int32_t act;                    // 1: leaky ReLU after the bias
    const uint16_t *slope;          // NULL, or multiply by the leaky ReLU derivative at the sign of this tensor
    int32_t sl_cs, sl_co;
    const uint16_t *add;            // NULL, or add this tensor
    int32_t ad_cs, ad_co;
    uint16_t *y;                    // BF16 output view, or
    int32_t y_cs, y_co;
    float *yf;                      // FP32 output (when y is NULL)
    int32_t yf_cs;
};

// A weight operand (B) of one product: 32 output channels x 16 input
// channels of one tap as the 64 lanes hold them (lane l: channel l mod 32,
// entries 8 (l / 32) .. + 7), 1 KB in a row: [phase][tile of 32 output
// channels][tap][16 input channels][lane][8].  Read from rows of a
// [output channel][tap][input channel] array, a load took 32 bytes from each
// of 32 cache lines.
__device__ inline bf16x8_t weight_operand(const ConvArgs &a, int ph, int ntile, int tap, int c, int lane)
{
    const int taps = a.k * a.k * a.k;
    const size_t f = ((size_t)(ph * (a.npad / 32) + ntile) * taps + tap) * (a.cin / 16) + c / 16;
    return ld8(a.w + f * 512 + (uint32_t)lane * 8u);
}

// Epilogue of one 32 x 32 tile of a wave (lane l: column n0 + l mod 32, rows
// 8 (v / 4) + 4 (l / 32) + v % 4): bias and leaky ReLU, or the leaky ReLU
// derivative and the second gradient, then the store.  The tile goes through
// the wave's own kTileWords words of LDS, so that a lane then holds 8
// channels of one row and the tensors are read and written 16 bytes at a time
// (channels come in multiples of 16); two bytes at a time, the epilogue took
// as long as the products.  position(row, op): the row's output position;
// false outside the grid; asked for rows lane / 4 and lane / 4 + 16, and with
// kF32 for others where the output is FP32.
constexpr int kTileRow = 40;   // words per row: rows 4 apart (a write's two halves) on different banks
constexpr int kTileWords = 32 * kTileRow;

template <bool kF32, typename F>
__device__ __forceinline__ void store_tile(const ConvArgs &a, float *tile, const f32x16_t &acc, int n0, int lane, F position)
{
    const int half = lane >> 5, r = lane & 31;
    const float bias = a.bias && n0 + r < a.cout ? a.bias[n0 + r] : 0.0f;
    __builtin_amdgcn_wave_barrier();   // the tile before has been read
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        float val = acc[v];
        if (a.bias) val += bias;
        if (a.act) val = val > 0.0f ? val : kLeak * val;
        tile[(8 * (v >> 2) + 4 * half + (v & 3)) * kTileRow + r] = val;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (kF32 && !a.y) {   // FP32 output: the tile's own columns, n0 .. min(n0 + 32, cout) - 1
        const int cols = min(32, a.cout - n0);   // (not above 0 where n0 is in the padding)
        for (int i = lane; i < 32 * cols; i += 64) {
            size_t op;
            if (position(i / cols, op)) a.yf[op * a.yf_cs + n0 + i % cols] = tile[(i / cols) * kTileRow + i % cols];
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (lane >> 2) + 16 * i, n = n0 + 8 * (lane & 3);
        size_t op;
        if (!position(row, op) || n >= a.cout) continue;
        float val[8];
        *reinterpret_cast<u32x4 *>(val) = *reinterpret_cast<const u32x4 *>(tile + row * kTileRow + 8 * (lane & 3));
        *reinterpret_cast<u32x4 *>(val + 4) = *reinterpret_cast<const u32x4 *>(tile + row * kTileRow + 8 * (lane & 3) + 4);
        uint16_t h[8];
        if (a.slope) {
            *reinterpret_cast<u32x4 *>(h) = *reinterpret_cast<const u32x4 *>(a.slope + op * a.sl_cs + a.sl_co + n);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (!(bf2f(h[j]) > 0.0f)) val[j] *= kLeak;
        }
        if (a.add) {
            *reinterpret_cast<u32x4 *>(h) = *reinterpret_cast<const u32x4 *>(a.add + op * a.ad_cs + a.ad_co + n);
#pragma unroll
            for (int j = 0; j < 8; ++j) val[j] += bf2f(h[j]);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) h[j] = f2bf(val[j]);
        *reinterpret_cast<u32x4 *>(a.y + op * a.y_cs + a.y_co + n) = *reinterpret_cast<const u32x4 *>(h);
    }
}

// The convolutions between levels: K = 2, stride 2 (down, and the gradient of
// up), one product over 8 taps; K = 1 with 8 output phases (up, and the
// gradient of down), 8 products of the same rows.  A wave owns 32 rows (input
// positions or pairs of them) x NT tiles of 32 columns of `phases`
// consecutive phases.  A phase is a chain of K^3 cin / 16 steps whose operands
// come straight from memory, D steps ahead in registers: there is no reuse to
// stage, and the chain's loads are all there is to wait for on small grids.
// The ring runs on into the next phase, so its operands arrive during the
// epilogue.  The input grid is K times the row grid, so all rows read are
// inside; rows past the end repeat the last and are not stored.
// Measured, 64^3, base 32, four levels: the three down and three up
// convolutions of one sample 116 us before (a step's loads waited for, a wave
// per 32 x 64 tile and phase), 52 now; the six gradients of four samples 250
// and 180, of which 120 is the level of 64^3, where the tensors' rows of 64
// bytes are half a cache line.
template <int NT, int K, int D>
__global__ __launch_bounds__(256) void conv_kernel(ConvArgs a, int32_t phases)
{
    __shared__ __attribute__((aligned(16))) float tiles[4][kTileWords];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int half = lane >> 5;
    const uint32_t mtot = (uint32_t)a.batch * a.mz * a.my * a.mx;
    const uint32_t tile = __builtin_amdgcn_readfirstlane((blockIdx.x * (blockDim.x >> 6) + wave) * 32u);
    const int n0 = blockIdx.y * 32 * NT;
    if (tile >= mtot) return;
    const auto row_at = [&](uint32_t m, int &qz, int &qy, int &qx) {
        uint32_t t = min(m, mtot - 1);
        qx = t % a.mx;
        t /= a.mx;
        qy = t % a.my;
        t /= a.my;
        qz = t % a.mz;
        return (int)(t / a.mz);
    };
    int qz, qy, qx;
    int b = row_at(tile + (lane & 31), qz, qy, qx);
    const uint16_t *const xrow =
        a.x + (size_t)(((b * a.iz + K * qz) * a.iy + K * qy) * a.ix + K * qx) * a.x_cs + a.x_co + 8 * half;
    // output positions (phase 0) of the two rows that this lane stores
    size_t op0[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        b = row_at(tile + (lane >> 2) + 16 * i, qz, qy, qx);
        op0[i] = (size_t)((b * a.oz + a.s_out * qz) * a.oy + a.s_out * qy) * a.ox + a.s_out * qx;
    }

    const int nc = a.cin / 16, steps = K * K * K * nc;
    const int ph_end = (blockIdx.z + 1) * phases;
    // the step that is loaded next: phase, tap, channels
    int lph = blockIdx.z * phases, tap = 0, c = 0, j = 0;
    bf16x8_t A[D], B[D][NT];
    const uint16_t *const wlane = a.w + (size_t)(n0 / 32) * steps * 512 + lane * 8;
    const size_t wphase = (size_t)(a.npad / 32) * steps * 512, wtile = (size_t)steps * 512;
    const auto load = [&](int d) {
        size_t at = c * 16;
        if (K == 2) at += (size_t)(((tap >> 2) * a.iy + ((tap >> 1) & 1)) * a.ix + (tap & 1)) * a.x_cs;
        A[d] = ld8(xrow + at);
#pragma unroll
        for (int s = 0; s < NT; ++s) B[d][s] = ld8(wlane + lph * wphase + s * wtile + (size_t)j * 512);
        if (j + 1 < steps) {
            ++j;
            if (++c == nc) c = 0, ++tap;
        } else if (lph + 1 < ph_end) {
            ++lph, tap = c = j = 0;
        }   // else: past the end, the last step again
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d);
    for (int ph = blockIdx.z * phases; ph < ph_end; ++ph) {
        f32x16_t acc[NT];
#pragma unroll
        for (int s = 0; s < NT; ++s)
            for (int v = 0; v < 16; ++v) acc[s][v] = 0.0f;
        for (int k = 0; k < steps; k += D)
#pragma unroll
            for (int d = 0; d < D; ++d) {
#pragma unroll
                for (int s = 0; s < NT; ++s)
                    acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[d], B[d][s], acc[s], 0, 0, 0);
                load(d);
            }
        const size_t shift = (size_t)(((ph >> 2) & 1) * a.oy + ((ph >> 1) & 1)) * a.ox + (ph & 1);
#pragma unroll
        for (int s = 0; s < NT; ++s)
            store_tile<false>(a, tiles[wave], acc[s], n0 + 32 * s, lane, [&](int row, size_t &op) {
                op = op0[row >> 4] + shift;
                return tile + row < mtot;
            });
    }
}

// 3^3 convolutions (stride 1, padding 1) -- most of the network's work --
// with the input staged in LDS.  A workgroup owns a brick of Z x 8 x 8 output
// positions and NC tiles of 32 columns; its 2 NC waves are the brick's two
// y-halves times the column tiles, and a wave computes Z 32-row tiles (4 x 8
// positions of one z-plane each) of its columns.  For every chunk of CC input
// channels the workgroup loads the (Z + 2) x 10 x 10 halo of the brick (zero
// outside the volume).
//
// A tap row (ty, tx) of one input plane is the A operand of up to three
// output planes (tz = 0, 1, 2), so a wave walks the input planes and reads
// each operand from LDS once for three products: (Z + 2) / (3 Z) reads per
// product.  The 27 weight operands of a chunk stay in registers; each is
// reloaded for the next chunk right after its last use, a chunk ahead of its
// next.  An output's products come in the order chunk, tz, ty, tx, channel,
// whatever Z.
//
// A halo position is 16 channels (32 bytes, two 16-byte units) and a halo
// row of 10 positions is padded to 21 units: the 16 lanes of an operand read
// that the LDS serves together (two x-rows of 8 positions) then fall on 16
// different units of a 256-byte window, the even ones for one row and the
// odd ones for the other, so the reads are free of bank conflicts.  Chunks
// of 32 channels are two such planes.
//
// Measured, one sample of 64^3, base 32, four levels (122 GFLOP, 0.11 ms at
// the rate of a large BF16 matrix product): forward 1.21 ms before (each
// operand read from LDS for one product, weights in rows, two-byte epilogue),
// 0.34 ms now.  What is left is the latency of a chunk on the small grids (a
// wave per SIMD or less) and, on the large ones, the halo loads between two
// barriers with two waves per SIMD, whose 256 registers are all taken (three
// are spilled in the form with two column tiles).
constexpr int kH3 = 10;                       // halo edge in y and x
constexpr int kRow3 = kH3 * 16 + 8;           // 168 elements per halo row: an odd number of 16-byte units

// kFull: the input channels are a multiple of CC (else the last chunk's second
// half is zero, and its weights are not there to be read).
template <int Z, int CC, int NC, bool kFull>
__global__ __launch_bounds__(128 * NC, Z >= 4 && CC == 16 ? 2 : 1) void conv3_kernel(ConvArgs a)
{
    constexpr int kThreads = 128 * NC, kHalf = CC / 16;
    constexpr int kPlane = (Z + 2) * kH3 * kRow3;                // elements of 16 channels of the halo
    // the halo's rows of 10 positions: kUnits 16-byte units each, kRowsAt
    // rows at a time
    constexpr int kUnits = kH3 * (CC / 8), kRows = (Z + 2) * kH3;
    constexpr int kRowsAt = kThreads / kUnits, kPer = (kRows + kRowsAt - 1) / kRowsAt;
    constexpr bool kAhead = Z < 4;   // few workgroups: the next halo is loaded during the products
    constexpr int kTiles = 2 * 2 * NC * kTileWords;   // the epilogue's tiles, in elements of the halo
    __shared__ __attribute__((aligned(16))) uint16_t halo[kHalf * kPlane > kTiles ? kHalf * kPlane : kTiles];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int half = lane >> 5;
    const int r = lane & 31;
    const int nbx = (a.mx + 7) / 8, nby = (a.my + 7) / 8, nbz = (a.mz + Z - 1) / Z;
    // neighbouring bricks share halos: consecutive ones on one XCD (its
    // workgroups are every eighth)
    int bid = blockIdx.x;
    if (gridDim.x % 8 == 0) bid = (bid % 8) * (gridDim.x / 8) + bid / 8;
    const int bxi = bid % nbx;
    bid /= nbx;
    const int byi = bid % nby;
    bid /= nby;
    const int bzi = bid % nbz;
    const int b = bid / nbz;
    const int z0 = bzi * Z, y0 = byi * 8, x0 = bxi * 8;
    const int n0 = (blockIdx.y * NC + (wave >> 1)) * 32;
    const int ly = (wave & 1) * 4 + (r >> 3), lx = r & 7;
    const uint16_t *const arow = halo + ly * kRow3 + lx * 16 + 8 * half;
    const int ntile = __builtin_amdgcn_readfirstlane(n0 / 32);
    const uint16_t *const wtile = a.w + (size_t)ntile * 27 * a.cin * 32;
    const auto weights = [&](int t, int c) { return ld8(wtile + (size_t)(t * (a.cin / 16) + c / 16) * 512 + (uint32_t)lane * 8u); };

    // this lane's unit of a halo row and its first row
    const int unit = tid % kUnits, row0 = tid / kUnits;
    const int hx = unit / (CC / 8), hg = unit % (CC / 8);
    const int xx = x0 + hx - 1;
    uint16_t *const hdst = halo + (hg >> 1) * kPlane + row0 * kRow3 + hx * 16 + 8 * (hg & 1);
    // Loads are unconditional, from the nearest position inside the volume,
    // and zeroed when stored: with branches around them the compiler cannot
    // count them and waits for every load in flight, the next weights too
    // (178 -> 171 us for four samples of 64^3 and 32 -> 64 channels).
    const auto load_row = [&](int first, int e, int c0) {
        const int row = first + kRowsAt * e;
        const int zz = min(max(z0 + row / kH3 - 1, 0), a.iz - 1), yy = min(max(y0 + row % kH3 - 1, 0), a.iy - 1);
        const int xc = min(max(xx, 0), a.ix - 1), c = min(c0 + 8 * hg, a.cin - 8);
        return *reinterpret_cast<const u32x4 *>(a.x + (size_t)(((b * a.iz + zz) * a.iy + yy) * a.ix + xc) * a.x_cs + a.x_co + c);
    };
    const auto store_row = [&](int first, int e, int c0, u32x4 v) {
        const int row = first + kRowsAt * e;
        const int zz = z0 + row / kH3 - 1, yy = y0 + row % kH3 - 1;
        const bool in = xx >= 0 && xx < a.ix && zz >= 0 && zz < a.iz && yy >= 0 && yy < a.iy && c0 + 8 * hg < a.cin;
        if (row0 < kRowsAt && row < kRows)
            *reinterpret_cast<u32x4 *>(hdst + kRowsAt * e * kRow3) = in ? v : u32x4{0u, 0u, 0u, 0u};
    };
    u32x4 ph[kAhead ? kPer : 1];
    const auto load_halo = [&](int c0) {
#pragma unroll
        for (int e = 0; e < kPer; ++e) ph[e] = load_row(row0, e, c0);
    };

    // (the loads come in the order of the loop's, halo before weights: what a
    // wait may leave in flight is the least over the ways that lead to it)
    if (kAhead) load_halo(0);
    __builtin_amdgcn_sched_barrier(0);
    f32x16_t acc[Z];
#pragma unroll
    for (int z = 0; z < Z; ++z)
        for (int v = 0; v < 16; ++v) acc[z][v] = 0.0f;
    bf16x8_t B[27][kHalf];
#pragma unroll
    for (int t = 0; t < 27; ++t) {
#pragma unroll
        for (int h = 0; h < kHalf; ++h) B[t][h] = kFull || h == 0 || a.cin > 16 ? weights(t, 16 * h) : zero8();
        __builtin_amdgcn_sched_barrier(0);
    }

    // products of one chunk; kNext: another one follows, its weights are loaded
    const auto chunk = [&](auto has_next, int c0) {
        constexpr bool kNext = decltype(has_next)::value;
        const int cn = c0 + CC;
        // operand (p, t) of the halo: input plane p, tap row and column t
        const auto operand = [&](int i, int h) {
            return ld8(arow + h * kPlane + ((i / 9) * kH3 + (i % 9) / 3) * kRow3 + (i % 3) * 16);
        };
        constexpr int kOps = 9 * (Z + 2);
        bf16x8_t A[3][kHalf];   // two operands are read ahead
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int h = 0; h < kHalf; ++h) A[i][h] = operand(i, h);
#pragma unroll
        for (int i = 0; i < kOps; ++i) {
            const int p = i / 9, t = i % 9;
            if (i + 2 < kOps)
#pragma unroll
                for (int h = 0; h < kHalf; ++h) A[(i + 2) % 3][h] = operand(i + 2, h);
#pragma unroll
            for (int tz = 0; tz < 3; ++tz) {
                const int z = p - tz;
                if (z < 0 || z >= Z) continue;
#pragma unroll
                for (int h = 0; h < kHalf; ++h)
                    acc[z] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[i % 3][h], B[9 * tz + t][h], acc[z], 0, 0, 0);
                if (kNext && z == Z - 1)
#pragma unroll
                    for (int h = 0; h < kHalf; ++h)
                        B[9 * tz + t][h] = kFull || h == 0 || cn + 16 < a.cin ? weights(9 * tz + t, cn + 16 * h) : zero8();
            }
            __builtin_amdgcn_sched_barrier(0);   // or the scheduler reads all operands at once and spills
        }
    };
    for (int c0 = 0; c0 < a.cin; c0 += CC) {
        lds_barrier();   // the previous chunk has been consumed
        if (kAhead) {
#pragma unroll
            for (int e = 0; e < kPer; ++e) store_row(row0, e, c0, ph[e]);
        } else {
            constexpr int kBatch = 5;   // rows in flight per lane
            int first = row0;           // as if new in every chunk: addresses kept from chunk to chunk would spill
            asm volatile("" : "+v"(first));
            static_assert(kAhead || kPer % kBatch == 0, "rows come in batches");
#pragma unroll
            for (int e0 = 0; e0 < kPer; e0 += kBatch) {
                u32x4 v[kBatch];
#pragma unroll
                for (int e = 0; e < kBatch; ++e) v[e] = load_row(first, e0 + e, c0);
#pragma unroll
                for (int e = 0; e < kBatch; ++e) store_row(first, e0 + e, c0, v[e]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        lds_barrier();
        if (c0 + CC < a.cin) {
            if (kAhead) load_halo(c0 + CC);
            __builtin_amdgcn_sched_barrier(0);
            chunk(std::true_type{}, c0);
        } else {
            chunk(std::false_type{}, c0);
        }
    }

    lds_barrier();   // the halo has been consumed: its LDS holds the tiles
    float *const tile = reinterpret_cast<float *>(halo) + wave * kTileWords;
#pragma unroll
    for (int z = 0; z < Z; ++z)
        store_tile<true>(a, tile, acc[z], n0, lane, [&](int i, size_t &op) {
            const int pz = z0 + z, py = y0 + (wave & 1) * 4 + (i >> 3), px = x0 + (i & 7);
            op = (size_t)((b * a.oz + pz) * a.oy + py) * a.ox + px;
            return pz < a.mz && py < a.my && px < a.mx;
        });
}

template <int CC, int NC, bool kFull>
static void launch_conv3_as(const ConvArgs &a, hipStream_t s)
{
    // z-planes per wave: four where that leaves a wave per SIMD, fewer on
    // smaller grids
    const int64_t yx = (int64_t)a.batch * ((a.my + 7) / 8) * ((a.mx + 7) / 8);
    const auto waves = [&](int Z) { return yx * ((a.mz + Z - 1) / Z) * 2 * (a.npad / 32); };
    const dim3 threads(128 * NC);
    const auto grid = [&](int Z) { return dim3((unsigned)(yx * ((a.mz + Z - 1) / Z)), (unsigned)(a.npad / (32 * NC)), 1); };
    if (CC == 16 && waves(4) >= 1024)
        hipLaunchKernelGGL((conv3_kernel<4, 16, NC, true>), grid(4), threads, 0, s, a);
    else if (waves(2) >= 1024)
        hipLaunchKernelGGL((conv3_kernel<2, CC, NC, kFull>), grid(2), threads, 0, s, a);
    else
        hipLaunchKernelGGL((conv3_kernel<1, CC, NC, kFull>), grid(1), threads, 0, s, a);
}

// ------------------------------------------------------------------ weight gradient
struct WgradArgs {
    const uint16_t *x;
    int32_t x_cs, x_co, x_c;        // forward input view (x_c channels present, multiple of 8)
    int32_t iz, iy, ix;
    int32_t mz, my, mx, batch;
    int32_t k, s_in, pad;
    int32_t nph, s_out, oz, oy, ox;
    const uint16_t *dy;             // gradient of the pre-activation output
    int32_t dy_cs, dy_co, dy_c;
    int32_t cin, cout;              // real channel counts (stored)
    uint32_t chunk;                 // rows per workgroup (multiple of 256)
    float *part;                    // [chunks][slots][cin][cout]
};

constexpr int kWgStep = 64;   // rows per wave and step

typedef short s16x4 __attribute__((ext_vector_type(4)));

// 4 positions (of row stride 32 channels) of the lane's channel, read
// transposed from a channels-last tile; p: see tr_lane.
__device__ inline uint2 tr_read4(const uint16_t *p)
{
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
    return __builtin_bit_cast(uint2, v);
}

// The lane's share of a transpose read's address.
__device__ inline int tr_lane(int lane)
{
    return ((lane & 15) >> 2) * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
}

// A wave stages its 64 rows of x and dy in LDS of its own, channels last, and
// reads the operands transposed (see wgrad3_kernel); the next 64 rows are
// loaded during the products.  Measured, 4 x 64^3, base 32, four levels: the six
// layers' kernels 216 us with the operands gathered two bytes at a time between
// two workgroup barriers, 156 now.
__global__ __launch_bounds__(256) void wgrad_kernel(WgradArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t xs[4][kWgStep][32];
    __shared__ __attribute__((aligned(16))) uint16_t ds[4][kWgStep][32];
    __shared__ float red[3][64][17];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int half = lane >> 5;
    const int r = lane & 31;
    const int ntile_o = (a.cout + 31) / 32;
    const int i0 = (blockIdx.y / ntile_o) * 32;
    const int o0 = (blockIdx.y % ntile_o) * 32;
    const int slot = blockIdx.z;
    const int tap = a.nph > 1 ? 0 : slot;
    const int ph = a.nph > 1 ? slot : 0;
    const int tz = tap / (a.k * a.k), ty = (tap / a.k) % a.k, tx = tap % a.k;
    const int ez = (ph >> 2) & 1, ey = (ph >> 1) & 1, ex = ph & 1;
    const uint32_t mtot = (uint32_t)a.batch * a.mz * a.my * a.mx;
    const uint32_t c_begin = blockIdx.x * a.chunk;
    const uint32_t c_end = min(c_begin + a.chunk, mtot);
    const int cg = (lane & 3) * 8;
    constexpr int kPer = kWgStep / 16;
    const bool x_in = i0 + cg < a.x_c, d_in = o0 + cg < a.dy_c;

    u32x4 vx[kPer], vd[kPer];
    bool in[kPer];
    const auto load = [&](uint32_t base) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const uint32_t m = base + wave * kWgStep + (lane >> 2) + 16 * j;
            in[j] = m < c_end;
            uint32_t t = min(m, c_end - 1);
            const int qx = t % a.mx;
            t /= a.mx;
            const int qy = t % a.my;
            t /= a.my;
            const int qz = t % a.mz;
            const int b = t / a.mz;
            // (no padding: the input grid is s_in times the row grid)
            const int zz = a.s_in * qz + tz, yy = a.s_in * qy + ty, xx = a.s_in * qx + tx;
            vx[j] = *reinterpret_cast<const u32x4 *>(
                a.x + (size_t)(((b * a.iz + zz) * a.iy + yy) * a.ix + xx) * a.x_cs + a.x_co + (x_in ? i0 + cg : 0));
            const size_t op = (size_t)((b * a.oz + a.s_out * qz + ez) * a.oy + a.s_out * qy + ey) * a.ox + a.s_out * qx + ex;
            vd[j] = *reinterpret_cast<const u32x4 *>(a.dy + op * a.dy_cs + a.dy_co + (d_in ? o0 + cg : 0));
        }
    };
    f32x16_t acc;
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    const uint16_t *const xr = &xs[wave][8 * half][0] + tr_lane(lane), *const dr = &ds[wave][8 * half][0] + tr_lane(lane);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    load(c_begin);
    for (uint32_t base = c_begin; base < c_end; base += 4 * kWgStep) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int rr = (lane >> 2) + 16 * j;
            *reinterpret_cast<u32x4 *>(&xs[wave][rr][cg]) = in[j] && x_in ? vx[j] : zero;
            *reinterpret_cast<u32x4 *>(&ds[wave][rr][cg]) = in[j] && d_in ? vd[j] : zero;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        load(min(base + 4 * kWgStep, c_end - 1));
#pragma unroll
        for (int kk = 0; kk < kPer; ++kk) {
            const uint2 a0 = tr_read4(xr + kk * 16 * 32), a1 = tr_read4(xr + (kk * 16 + 4) * 32);
            const uint2 b0 = tr_read4(dr + kk * 16 * 32), b1 = tr_read4(dr + (kk * 16 + 4) * 32);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, u32x4{a0.x, a0.y, a1.x, a1.y}),
                                                          __builtin_bit_cast(bf16x8_t, u32x4{b0.x, b0.y, b1.x, b1.y}), acc, 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();   // the rows have been read
    }
    // reduce the four waves' tiles in a fixed order
    if (wave > 0)
        for (int v = 0; v < 16; ++v) red[wave - 1][lane][v] = acc[v];
    lds_barrier();
    if (wave == 0) {
        for (int w = 0; w < 3; ++w)
            for (int v = 0; v < 16; ++v) acc[v] += red[w][lane][v];
        const int slots = a.nph > 1 ? a.nph : a.k * a.k * a.k;
        float *out = a.part + ((size_t)blockIdx.x * slots + slot) * a.cin * a.cout;
        for (int v = 0; v < 16; ++v) {
            const int i = i0 + 8 * (v >> 2) + 4 * half + (v & 3);
            const int o = o0 + r;
            if (i < a.cin && o < a.cout) out[(size_t)i * a.cout + o] = acc[v];
        }
    }
}

// Weight gradients of 3^3 convolutions, all 27 taps per workgroup.  The
// workgroup owns a 32 x 32 (input, output channel) tile and a chunk of
// 2 x 8 x 8 position bricks; per brick it stages dy and the 4 x 10 x 10
// input halo in LDS as they are in memory, channels last (one 16-byte
// write per 8 channels of a position).  The MFMA reduction runs over
// positions: one K-step is 16 positions (two x-rows of 8).  Its operands
// need 8 positions of one channel per lane, which the LDS transpose read
// (ds_read_b64_tr_b16) delivers from the channels-last tiles: within each
// group of 16 lanes, lane s gives the address of 4 channels (4 (s mod 4)
// onwards) at position s / 4, and lane i receives channel i at the 4
// positions.
//
// Three such reads hold the 10 positions of an input row, and the operands
// of its three x-taps are made from them in registers (the middle one by
// 16-bit shifts); the row of y-tap 2 is y-tap 0's of the next K-step.  The
// 27 taps are split over four waves, one per SIMD: wave w < 3 takes z-tap w's
// first 7 in (y, x) order, wave 3 the last two x-taps of y-tap 2 of every
// z-tap (6).  A chunk's bricks go up in z, so that two of a brick's four halo
// planes are the last one's and stay in LDS.  The next brick's loads are made
// during the products, from the nearest position inside the volume and zeroed
// when stored (see conv3_kernel).
//
// Measured, 4 x 64^3 positions, 32 x 32 channels (58 GFLOP, 52 us at the rate
// of a large BF16 matrix product): 110 us before (three waves of 9 taps, two
// reads per operand, bricks along x with whole halos, dy loaded when staged),
// 64 now; the 16 layers of a gradient of base 32, four levels 1090 and 710.
// Without the products it is 39, of which the partial sums' stores (56 MB)
// take a third.
constexpr int kGZ = 2, kGY = 8, kGX = 8;                 // brick
constexpr int kGHZ = kGZ + 2, kGHY = kGY + 2, kGHX = 12;  // halo (x padded from 10 to three reads)

// An input row: 10 positions of the lane's channel, and its x-taps.
struct TapRow { u32x4 v; uint32_t last; };

__device__ inline TapRow tap_row(const uint16_t *p)
{
    const uint2 r0 = tr_read4(p), r1 = tr_read4(p + 4 * 32);
    return {u32x4{r0.x, r0.y, r1.x, r1.y}, tr_read4(p + 8 * 32).x};
}

template <int TX>
__device__ inline bf16x8_t tap_operand(const TapRow &t)
{
    const auto mid = [](uint32_t hi, uint32_t lo) { return __builtin_amdgcn_alignbit(hi, lo, 16); };
    u32x4 v = t.v;
    if (TX == 1) v = u32x4{mid(v[1], v[0]), mid(v[2], v[1]), mid(v[3], v[2]), mid(t.last, v[3])};
    if (TX == 2) v = u32x4{v[1], v[2], v[3], t.last};
    return __builtin_bit_cast(bf16x8_t, v);
}

__global__ __launch_bounds__(256, 2) void wgrad3_kernel(WgradArgs a)
{
    constexpr int kThreads = 256, kXWords = kGHZ * kGHY * kGHX * 32;
    __shared__ __attribute__((aligned(16))) uint16_t xL[kXWords];                // 30 KB, [hz][hy][hx][ch]
    __shared__ __attribute__((aligned(16))) uint16_t dL[kGZ * kGY * kGX * 32];   // 8 KB, [lz][ly][lx][ch]
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    const int r = lane & 31;
    const int ntile_o = (a.cout + 31) / 32;
    const int i0 = (blockIdx.y / ntile_o) * 32;
    const int o0 = (blockIdx.y % ntile_o) * 32;
    const int nbx = (a.mx + kGX - 1) / kGX, nby = (a.my + kGY - 1) / kGY, nbz = (a.mz + kGZ - 1) / kGZ;
    const uint32_t nb = (uint32_t)a.batch * nbz * nby * nbx;
    // neighbouring columns share halos: consecutive chunks on one XCD
    uint32_t chunk = blockIdx.x;
    if (gridDim.x % 8 == 0) chunk = (chunk % 8) * (gridDim.x / 8) + chunk / 8;
    const uint32_t b_begin = chunk * a.chunk, b_end = min(b_begin + a.chunk, nb);

    // workgroups of the first input-channel tile also sum dy per output
    // channel (the bias gradient): a thread adds the 8 channels of the
    // positions that it stages
    const bool want_bias = i0 == 0;
    float bsum[8];
    for (int j = 0; j < 8; ++j) bsum[j] = 0.0f;

    // 16-byte items: two halo planes or a dy tile; thread t's are t, t + 256,
    // ...: all of one channel group g
    constexpr int kDyPer = kGZ * kGY * kGX * 4 / kThreads, kHaloItems = 2 * kGHY * 10 * 4;
    constexpr int kHaloPer = (kHaloItems + kThreads - 1) / kThreads;
    const int g = tid & 3;
    const bool x_in = i0 + 8 * g < a.x_c, d_in = o0 + 8 * g < a.dy_c;
    const uint16_t *const xg = a.x + a.x_co + (x_in ? i0 + 8 * g : 0);
    const uint16_t *const dg = a.dy + a.dy_co + (d_in ? o0 + 8 * g : 0);
    u32x4 ph[kHaloPer], pd[kDyPer];
    uint32_t h_in = 0, dy_in = 0;   // items inside the volume
    struct Brick { int b, bz, y0, x0; };
    const auto brick = [&](uint32_t t) {
        const int bz = t % nbz;
        t /= nbz;
        const int x0 = (int)(t % nbx) * kGX;
        t /= nbx;
        return Brick{(int)(t / nby), bz, (int)(t % nby) * kGY, x0};
    };
    const auto load_planes = [&](const Brick &k, int pair) {
        h_in = 0;
#pragma unroll
        for (int j = 0; j < kHaloPer; ++j) {
            const int pos = (tid + kThreads * j) >> 2, row = pos / 10;
            const int zz = k.bz * kGZ + 2 * pair + row / kGHY - 1, yy = k.y0 + row % kGHY - 1, xx = k.x0 + pos % 10 - 1;
            h_in |= (uint32_t)(x_in & ((uint32_t)zz < (uint32_t)a.iz) & ((uint32_t)yy < (uint32_t)a.iy) & ((uint32_t)xx < (uint32_t)a.ix)) << j;
            const int zc = min(max(zz, 0), a.iz - 1), yc = min(max(yy, 0), a.iy - 1), xc = min(max(xx, 0), a.ix - 1);
            ph[j] = *reinterpret_cast<const u32x4 *>(xg + (size_t)(((k.b * a.iz + zc) * a.iy + yc) * a.ix + xc) * a.x_cs);
        }
    };
    const auto load_dy = [&](const Brick &k) {
        dy_in = 0;
#pragma unroll
        for (int j = 0; j < kDyPer; ++j) {
            const int pos = (tid + kThreads * j) >> 2;
            const int zz = k.bz * kGZ + (pos >> 6), yy = k.y0 + ((pos >> 3) & 7), xx = k.x0 + (pos & 7);
            dy_in |= (uint32_t)(d_in & (zz < a.mz) & (yy < a.my) & (xx < a.mx)) << j;
            pd[j] = *reinterpret_cast<const u32x4 *>(
                dg + (size_t)(((k.b * a.oz + min(zz, a.oz - 1)) * a.oy + min(yy, a.oy - 1)) * a.ox + min(xx, a.ox - 1)) * a.dy_cs);
        }
    };
    constexpr int kPlane = kGHY * kGHX * 32;
    // halo planes 0, 1 (pair 0) and 2, 3 of brick bz: a pair keeps its place
    // when it becomes the next brick's first
    const auto place = [&](int bz, int plane) { return (((plane >> 1) ^ bz) & 1) * 2 + (plane & 1); };
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const auto store_planes = [&](int bz, int pair) {
        uint16_t *const to = xL + place(bz, 2 * pair) * kPlane + 8 * g;
#pragma unroll
        for (int j = 0; j < kHaloPer; ++j) {
            const int e = tid + kThreads * j, pos = e >> 2;
            if (e < kHaloItems)
                *reinterpret_cast<u32x4 *>(to + ((pos / 10) * kGHX + pos % 10) * 32) = (h_in >> j) & 1 ? ph[j] : zero;
        }
    };

    // the products of one brick; xz: the planes of z-taps
    const int x_lane = tr_lane(lane) + half * kGHX * 32;
    const uint16_t *const dw = dL + tr_lane(lane) + half * kGX * 32;
    constexpr int kSteps = kGZ * kGY / 2;
    const auto x_at = [&](const uint16_t *plane, int i, int ty) {   // K-step i
        return tap_row(plane + (2 * (i % (kGY / 2)) + ty) * kGHX * 32);
    };
    const auto dy_at = [&](int i) {
        const uint16_t *const p = dw + i * 2 * kGX * 32;
        const uint2 b0 = tr_read4(p), b1 = tr_read4(p + 4 * 32);
        return __builtin_bit_cast(bf16x8_t, u32x4{b0.x, b0.y, b1.x, b1.y});
    };
    const auto mma = [](bf16x8_t A, bf16x8_t B, f32x16_t c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, B, c, 0, 0, 0); };
    // Rows are read one ahead; the scheduling barriers keep the reads before
    // the products that hide them, and further ones from being hoisted.
    const auto stage = [&](auto products) {
        load_planes(brick(b_begin), 0);
        for (uint32_t bi = b_begin; bi < b_end; ++bi) {
            const Brick k = brick(bi), n = brick(min(bi + 1, b_end - 1));
            lds_barrier();   // the previous brick has been consumed
            if (bi == b_begin || k.bz == 0) {   // a column's first: nothing is there yet
                if (bi != b_begin) load_planes(k, 0);
                store_planes(k.bz, 0);
                load_planes(k, 1);
                load_dy(k);
            }
            store_planes(k.bz, 1);
#pragma unroll
            for (int j = 0; j < kDyPer; ++j) {
                const u32x4 v = (dy_in >> j) & 1 ? pd[j] : zero;
                *reinterpret_cast<u32x4 *>(&dL[((tid + kThreads * j) >> 2) * 32 + 8 * g]) = v;
                if (want_bias)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        bsum[2 * w] += bf2f((uint16_t)(v[w] & 0xffffu));
                        bsum[2 * w + 1] += bf2f((uint16_t)(v[w] >> 16));
                    }
            }
            lds_barrier();
            load_planes(n, 1);
            load_dy(n);
            __builtin_amdgcn_sched_barrier(0);
            products(k.bz);
        }
    };
    float *out = a.part + (size_t)chunk * ((size_t)27 * a.cin * a.cout + a.cout);
    const auto store = [&](const f32x16_t &acc, int tap) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {   // rows = input channels, columns = output channels
            const int i = i0 + 8 * (v >> 2) + 4 * half + (v & 3);
            const int o = o0 + r;
            if (i < a.cin && o < a.cout) out[((size_t)tap * a.cin + i) * a.cout + o] = acc[v];
        }
    };
    // (each kind of wave has the whole loop, with as many barriers, to itself:
    // with one loop around both, each kept accumulators of its own)
    if (wave < 3) {
        f32x16_t acc[7];
#pragma unroll
        for (int q = 0; q < 7; ++q)
            for (int v = 0; v < 16; ++v) acc[q][v] = 0.0f;
        stage([&](int bz) {
            const uint16_t *const xz[2] = {xL + x_lane + place(bz, wave) * kPlane, xL + x_lane + place(bz, wave + 1) * kPlane};
            TapRow t = x_at(xz[0], 0, 0), n;
            bf16x8_t B = dy_at(0);
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                n = x_at(xz[i / (kGY / 2)], i, 1);
                __builtin_amdgcn_sched_barrier(0);
                acc[0] = mma(tap_operand<0>(t), B, acc[0]);
                acc[1] = mma(tap_operand<1>(t), B, acc[1]);
                acc[2] = mma(tap_operand<2>(t), B, acc[2]);
                __builtin_amdgcn_sched_barrier(0);
                t = x_at(xz[i / (kGY / 2)], i, 2);
                __builtin_amdgcn_sched_barrier(0);
                acc[3] = mma(tap_operand<0>(n), B, acc[3]);
                acc[4] = mma(tap_operand<1>(n), B, acc[4]);
                acc[5] = mma(tap_operand<2>(n), B, acc[5]);
                __builtin_amdgcn_sched_barrier(0);
                const int k = min(i + 1, kSteps - 1);
                const bool plane = k % (kGY / 2) == 0;   // a new z-plane: no row in common
                if (plane) n = x_at(xz[k / (kGY / 2)], k, 0);
                const bf16x8_t next = dy_at(k);
                __builtin_amdgcn_sched_barrier(0);
                acc[6] = mma(tap_operand<0>(t), B, acc[6]);
                if (plane) t = n;
                B = next;
                __builtin_amdgcn_sched_barrier(0);
            }
        });
#pragma unroll
        for (int q = 0; q < 7; ++q) store(acc[q], 9 * wave + q);
    } else {
        f32x16_t acc[6];
#pragma unroll
        for (int q = 0; q < 6; ++q)
            for (int v = 0; v < 16; ++v) acc[q][v] = 0.0f;
        stage([&](int bz) {
            const uint16_t *xz[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) xz[p] = xL + x_lane + place(bz, p) * kPlane;
            TapRow t = x_at(xz[0], 0, 2), n;
            bf16x8_t B = dy_at(0);
#pragma unroll
            for (int i = 0; i < kSteps; ++i) {
                const int k = min(i + 1, kSteps - 1);
                bf16x8_t next = B;
#pragma unroll
                for (int tz = 0; tz < 3; ++tz) {
                    n = tz < 2 ? x_at(xz[i / (kGY / 2) + tz + 1], i, 2) : x_at(xz[k / (kGY / 2)], k, 2);
                    if (tz == 2) next = dy_at(k);
                    __builtin_amdgcn_sched_barrier(0);
                    acc[2 * tz] = mma(tap_operand<1>(t), B, acc[2 * tz]);
                    acc[2 * tz + 1] = mma(tap_operand<2>(t), B, acc[2 * tz + 1]);
                    t = n;
                    __builtin_amdgcn_sched_barrier(0);
                }
                B = next;
            }
        });
#pragma unroll
        for (int q = 0; q < 6; ++q) store(acc[q], 9 * (q >> 1) + 7 + (q & 1));
    }
    // bias partials of this chunk, after all weight partials: the 16 lanes of
    // a wave with the same channel group, then the four waves
    if (want_bias) {
        float *const bred = reinterpret_cast<float *>(xL);   // [4][32]
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int off = 4; off < 64; off <<= 1) bsum[j] += __shfl_xor(bsum[j], off, 64);
        lds_barrier();
        if (lane < 4)
#pragma unroll
            for (int j = 0; j < 8; ++j) bred[wave * 32 + 8 * lane + j] = bsum[j];
        lds_barrier();
        if (tid < 32 && o0 + tid < a.cout) {
            const size_t row = (size_t)27 * a.cin * a.cout + a.cout;   // a chunk's weight partials, then its bias partials
            a.part[(size_t)chunk * row + (size_t)27 * a.cin * a.cout + o0 + tid] =
                (bred[tid] + bred[32 + tid]) + (bred[64 + tid] + bred[96 + tid]);
        }
    }
}

// Sum the chunk partials: g[e] = sum_c part[c][e].  A workgroup takes 32
// consecutive elements; its 8 chunk lanes sum the chunks c = lane mod 8 and
// are then added in lane order, so the result does not depend on timing.  Eight
// chunks are loaded at a time: one after the other, 512 chunks of a bias took
// 16 us, now 5, and the 23 sums of a gradient of base 32, four levels 370 and 230.
constexpr int kSumElems = 32, kSumLanes = 8;

__global__ __launch_bounds__(256) void sum_chunks_kernel(const float *part, int32_t chunks, int64_t n, float *g)
{
    __shared__ float red[kSumLanes][kSumElems + 1];
    const int ex = threadIdx.x % kSumElems, cl = threadIdx.x / kSumElems;
    const int64_t e = (int64_t)blockIdx.x * kSumElems + ex;
    float s = 0.0f;
    if (e < n) {
        int c = cl;
        for (; c + 7 * kSumLanes < chunks; c += 8 * kSumLanes) {   // eight loads in flight, added in order
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = part[(size_t)(c + k * kSumLanes) * n + e];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += v[k];
        }
        for (; c < chunks; c += kSumLanes) s += part[(size_t)c * n + e];
    }
    red[cl][ex] = s;
    __syncthreads();
    if (cl == 0 && e < n) {
        float t = 0.0f;
        for (int k = 0; k < kSumLanes; ++k) t += red[k][ex];
        g[e] = t;
    }
}

// Column sums of a channels-last BF16 view over npos positions (bias
// gradients): partial[block][c], then a fixed-order sum.  A thread adds 8
// channels (16 bytes) of every rows-th position of its block's part; read 2
// bytes at a time, 4 x 64^3 positions of 32 channels took 77 us, now 23 (67 MB
// in half cache lines; 14 us at the rate of a large copy).
constexpr int kColBlocks = 512;

__global__ __launch_bounds__(256) void colsum_kernel(const uint16_t *x, int32_t cs, int32_t co, int32_t C,
                                                     uint32_t npos, float *part)
{
    __shared__ float red[8][256];
    const uint32_t per = (npos + gridDim.x - 1) / gridDim.x;
    const uint32_t p0 = min(blockIdx.x * per, npos), p1 = min(p0 + per, npos);
    const int all = C / 8;   // channel groups (channels come in multiples of 16)
    for (int g0 = 0; g0 < all; g0 += 256) {
        const int groups = min(all - g0, 256), rows = 256 / groups;
        const int g = threadIdx.x % groups, sub = threadIdx.x / groups;
        float s[8];
        for (int j = 0; j < 8; ++j) s[j] = 0.0f;
        if (sub < rows) {
            const uint16_t *const xg = x + co + 8 * (g0 + g);
#pragma unroll 4
            for (uint32_t p = p0 + sub; p < p1; p += rows) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(xg + (size_t)p * cs);
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    s[2 * w] += bf2f((uint16_t)(v[w] & 0xffffu));
                    s[2 * w + 1] += bf2f((uint16_t)(v[w] >> 16));
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) red[j][threadIdx.x] = s[j];
        __syncthreads();
        for (int c = threadIdx.x; c < 8 * groups; c += 256) {
            float t = 0.0f;
            for (int q = 0; q < rows; ++q) t += red[c & 7][q * groups + (c >> 3)];
            part[(size_t)blockIdx.x * C + 8 * g0 + c] = t;
        }
    }
}

// ------------------------------------------------------------------ elementwise
// Weight layouts for the GEMMs from the FP32 master weights W[slot][cin][cout]:
//   operands (ph, n, t, c) as weight_operand has them, with slot = ph (phase
//   layouts) or t (flipped: T-1-t), value W[slot][c][n] (forward) or
//   W[slot][n][c] (transposed, backward-data).
struct PrepArgs {
    const float *W;
    int32_t cin, cout, nslots;
    uint16_t *out;
    int32_t nph, taps, npad, crow;
    int32_t transposed, flip;
};

// Every layout job of the network in one launch: blockIdx.y is the job,
// the x dimension strides over its elements.
__global__ void prep_weights_kernel(const PrepArgs *jobs)
{
    const PrepArgs a = jobs[blockIdx.y];
    const int64_t total = (int64_t)a.nph * a.npad * a.taps * a.crow;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int lane = (e >> 3) & 63;
        int64_t t = e >> 9;
        const int c = 16 * (int)(t % (a.crow / 16)) + 8 * (lane >> 5) + (int)(e & 7);
        t /= a.crow / 16;
        const int tap = t % a.taps;
        t /= a.taps;
        const int n = 32 * (int)(t % (a.npad / 32)) + (lane & 31);
        const int ph = t / (a.npad / 32);
        const int slot = a.nph > 1 ? ph : (a.flip ? a.nslots - 1 - tap : tap);
        float v = 0.0f;
        if (a.transposed) {
            if (n < a.cin && c < a.cout) v = a.W[((size_t)slot * a.cin + n) * a.cout + c];
        } else {
            if (c < a.cin && n < a.cout) v = a.W[((size_t)slot * a.cin + c) * a.cout + n];
        }
        a.out[e] = f2bf(v);
    }
}

// FP32 [npos][c] -> BF16 [npos][cpad], zero padded; a thread writes 8 channels.
__global__ void to_bf16_padded_kernel(const float *x, int32_t c, int32_t cpad, int64_t npos, uint16_t *out)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t groups = cpad / 8;
    if (e >= npos * groups) return;
    const int64_t p = e / groups;
    const int c0 = 8 * (int)(e % groups);
    uint16_t h[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) h[j] = c0 + j < c ? f2bf(x[p * c + c0 + j]) : (uint16_t)0;
    *reinterpret_cast<u32x4 *>(out + e * 8) = *reinterpret_cast<const u32x4 *>(h);
}

// dy = 2 (y - t) / count, and per-block FP64 partial sums of (y - t)^2.
__global__ __launch_bounds__(256) void mse_kernel(const float *y, const float *t, int64_t count, float *dy,
                                                  double *part)
{
    __shared__ double red[256];
    double s = 0.0;
    const float scale = (float)(2.0 / (double)count);
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x) {
        const float d = y[e] - t[e];
        s += (double)d * d;
        if (dy) dy[e] = scale * d;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// One workgroup of 256: every 256th value per thread, then a tree.
__global__ __launch_bounds__(256) void sum_f64_kernel(const double *part, int32_t n, double *out)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

__global__ void adam_kernel(float *p, const float *g, float *m, float *v, int64_t n, float lr_t, float b1, float b2,
                            float eps)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const float ge = g[e];
    const float me = b1 * m[e] + (1.0f - b1) * ge;
    const float ve = b2 * v[e] + (1.0f - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    p[e] -= lr_t * me / (sqrtf(ve) + eps);
}

// He-normal initialisation from a counter hash (splitmix64) and Box-Muller.
__device__ inline uint64_t splitmix64(uint64_t z)
{
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void init_normal_kernel(float *p, int64_t n, float stddev, uint64_t seed, int64_t offset)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const uint64_t h = splitmix64(seed ^ splitmix64((uint64_t)(offset + e)));
    const double u1 = ((h >> 11) + 0.5) * (1.0 / 9007199254740992.0);
    const double u2 = ((splitmix64(h) >> 11) + 0.5) * (1.0 / 9007199254740992.0);
    p[e] = (float)(stddev * sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
}

__global__ void fill_f32_kernel(float *p, int64_t n, float v)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = v;
}

__global__ void fill_u16_kernel(uint16_t *p, int64_t n)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) p[e] = 0;
}

inline unsigned nblk(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// ------------------------------------------------------------------ runtime
namespace {

int32_t round_up(int32_t v, int32_t m) { return (v + m - 1) / m * m; }
int32_t npad_for(int32_t rows) { return rows >= 64 ? round_up(rows, 64) : round_up(rows, 32); }
int taps_of(Layer::Kind k) { return k == Layer::CONV3 ? 27 : 8; }

}  // namespace

int64_t Net::positions(int level, int32_t n) const
{
    return (int64_t)n * (nz_ >> level) * (ny_ >> level) * (nx_ >> level);
}

// Split-K plan of a layer's weight gradient for a batch of n: 3^3 layers
// reduce bricks of 2 x 8 x 8 positions with all 27 taps per workgroup
// (about 512 workgroups in all); the other kinds reduce rows per tap with
// the generic kernel (about 4096 workgroups).  chunks x taps x cin x cout
// partial sums are written.
Net::WgradPlan Net::plan_wgrad(const Layer &L, int32_t n) const
{
    WgradPlan p;
    const int64_t ctiles = (int64_t)((L.cin + 31) / 32) * ((L.cout + 31) / 32);
    if (L.kind == Layer::CONV3) {
        const int l = L.level_out;
        const int64_t nb = (int64_t)n * (((nz_ >> l) + kGZ - 1) / kGZ) * (((ny_ >> l) + kGY - 1) / kGY) *
                           (((nx_ >> l) + kGX - 1) / kGX);
        // about 512 workgroups in all: two per CU resident at once, one round
        // (measured 4 x 64^3, base 32, four levels, with the sums of the
        // partials: 1.13 ms; 256: 1.19, 384: 1.23, 768: 1.41, 1024: 1.50)
        int64_t chunks = std::min<int64_t>(nb, std::max<int64_t>(1, 512 / ctiles));
        p.most = chunks;
        p.chunk = (uint32_t)((nb + chunks - 1) / chunks);
        p.chunks = (nb + p.chunk - 1) / p.chunk;
        p.bricks = true;
    } else {
        const int64_t rows = L.kind == Layer::UP2 ? positions(L.level_in, n) : positions(L.level_out, n);
        const int64_t tiles = ctiles * taps_of(L.kind);
        int64_t chunks = std::min<int64_t>((rows + 1023) / 1024, std::max<int64_t>(1, 4096 / tiles));
        p.most = chunks;
        uint32_t chunk = (uint32_t)((rows + chunks - 1) / chunks);
        p.chunk = (chunk + 255) / 256 * 256;
        p.chunks = (rows + p.chunk - 1) / p.chunk;
        p.bricks = false;
    }
    return p;
}

// The forward and backward-data layout jobs of every layer.
static std::vector<PrepArgs> prep_jobs(const std::vector<Layer> &layers, float *params)
{
    std::vector<PrepArgs> jobs;
    for (const auto &L : layers) {
        const int taps = taps_of(L.kind);
        PrepArgs f{params + L.w_off, L.cin, L.cout, taps, L.wf, 1, taps, L.npad_f, L.cin_buf, 0, 0};
        PrepArgs b{params + L.w_off, L.cin, L.cout, taps, L.wb, 1, taps, L.npad_b, L.cout_buf, 1, 0};
        if (L.kind == Layer::CONV3) {
            b.flip = 1;
        } else if (L.kind == Layer::UP2) {
            f.nph = 8;   // forward: eight phase GEMMs over the input channels
            f.taps = 1;
        } else {
            b.nph = 8;   // down2 backward-data: eight phase GEMMs
            b.taps = 1;
        }
        jobs.push_back(f);
        jobs.push_back(b);
    }
    return jobs;
}

Net::Status Net::create(int dev, int32_t cin, int32_t cout, int32_t base, int32_t levels, int32_t nmax, int32_t nz,
                        int32_t ny, int32_t nx, uint64_t seed, hipStream_t s)
{
    device = dev;
    if (cin < 1 || cout < 1 || base < 16 || base % 16 || levels < 1 || levels > 6 || nmax < 1 || nz < 1 || ny < 1 ||
        nx < 1)
        return {BAD_SHAPE, "bad network shape (base must be a positive multiple of 16, 1 <= levels <= 6)"};
    const int32_t div = 1 << (levels - 1);
    if (nz % div || ny % div || nx % div) return {BAD_SHAPE, "grid dimensions must be divisible by 2^(levels-1)"};
    if ((int64_t)nmax * nz * ny * nx >= (1ll << 31)) return {BAD_SHAPE, "batch x cells must stay below 2^31"};
    if ((int64_t)base << (levels - 1) > 4096) return {BAD_SHAPE, "more than 4096 channels"};
    cin_ = cin;
    cout_ = cout;
    base_ = base;
    levels_ = levels;
    nmax_ = nmax;
    nz_ = nz;
    ny_ = ny;
    nx_ = nx;
    cin_pad_ = round_up(cin, 16);
    cout_pad_ = round_up(cout, 16);
    std::vector<int32_t> ch(levels);
    for (int l = 0; l < levels; ++l) ch[l] = base << l;

    // layers in parameter order
    auto add = [&](Layer::Kind k, const std::string &name, int32_t ci, int32_t co, int32_t ci_buf, int32_t co_buf,
                   int lin, int lout) {
        Layer L;
        L.kind = k;
        L.name = name;
        L.cin = ci;
        L.cout = co;
        L.cin_buf = ci_buf;
        L.cout_buf = co_buf;
        L.level_in = lin;
        L.level_out = lout;
        L.nw = (int64_t)taps_of(k) * ci * co;
        L.w_off = nparam_;
        L.b_off = nparam_ + L.nw;
        nparam_ += L.nw + co;
        layers_.push_back(L);
    };
    int32_t c = cin;
    int32_t cbuf = cin_pad_;
    for (int l = 0; l < levels; ++l) {
        add(Layer::CONV3, "e" + std::to_string(l) + "a", c, ch[l], cbuf, ch[l], l, l);
        add(Layer::CONV3, "e" + std::to_string(l) + "b", ch[l], ch[l], ch[l], ch[l], l, l);
        if (l < levels - 1) {
            add(Layer::DOWN2, "d" + std::to_string(l), ch[l], ch[l + 1], ch[l], ch[l + 1], l, l + 1);
            c = cbuf = ch[l + 1];
        }
    }
    for (int l = levels - 2; l >= 0; --l) {
        add(Layer::UP2, "u" + std::to_string(l), ch[l + 1], ch[l], ch[l + 1], ch[l], l + 1, l);
        add(Layer::CONV3, "q" + std::to_string(l) + "a", 2 * ch[l], ch[l], 2 * ch[l], ch[l], l, l);
        add(Layer::CONV3, "q" + std::to_string(l) + "b", ch[l], ch[l], ch[l], ch[l], l, l);
    }
    add(Layer::CONV3, "out", ch[0], cout, ch[0], cout_pad_, 0, 0);

    auto alloc = [&](size_t bytes) -> void * {
        void *p = nullptr;
        if (hipMalloc(&p, bytes < 256 ? 256 : bytes) != hipSuccess) return nullptr;
        allocs_.push_back(p);
        return p;
    };
#define ALLOC(ptr, type, count)                                              \
    do {                                                                     \
        ptr = (type *)alloc(sizeof(type) * (size_t)(count));                 \
        if (!ptr) return {NO_MEMORY, "device allocation failed"};          \
    } while (0)

    ALLOC(d_params_, float, nparam_);
    ALLOC(d_grads_, float, nparam_);
    ALLOC(d_m_, float, nparam_);
    ALLOC(d_v_, float, nparam_);
    for (auto &L : layers_) {
        const int taps = taps_of(L.kind);
        L.npad_f = npad_for(L.cout);
        L.npad_b = npad_for(L.cin);
        // forward: conv3 and down2 are tap GEMMs, up2 is a phase GEMM; backward the other way round
        ALLOC(L.wf, uint16_t, (size_t)L.npad_f * taps * L.cin_buf);
        ALLOC(L.wb, uint16_t, (size_t)L.npad_b * taps * L.cout_buf);
    }
    ALLOC(d_loss_part_, double, 1024 + 1);
    ALLOC(d_xin_, uint16_t, positions(0, nmax) * cin_pad_);
    ALLOC(d_gy_, uint16_t, positions(0, nmax) * cout_pad_);
    ha_.assign(levels, nullptr);
    cat_.assign(levels, nullptr);
    hd_.assign(levels, nullptr);
    hqa_.assign(levels, nullptr);
    hqb_.assign(levels, nullptr);
    g1_.assign(levels, nullptr);
    g2_.assign(levels, nullptr);
    gcat_.assign(levels, nullptr);
    for (int l = 0; l < levels; ++l) {
        const int64_t P = positions(l, nmax);
        ALLOC(ha_[l], uint16_t, P * ch[l]);
        ALLOC(g1_[l], uint16_t, P * ch[l]);
        ALLOC(g2_[l], uint16_t, P * ch[l]);
        if (l > 0) ALLOC(hd_[l], uint16_t, P * ch[l]);
        if (l < levels - 1) {
            ALLOC(cat_[l], uint16_t, P * 2 * ch[l]);
            ALLOC(gcat_[l], uint16_t, P * 2 * ch[l]);
            ALLOC(hqa_[l], uint16_t, P * ch[l]);
            ALLOC(hqb_[l], uint16_t, P * ch[l]);
        }
    }
    ALLOC(hbot_, uint16_t, positions(levels - 1, nmax) * ch[levels - 1]);
    // split-K partials: the largest chunks x taps x cin x cout of any layer and
    // batch.  The chunks of a plan may be fewer with a larger batch (512 for
    // 512 bricks, 384 of two for 768); the limit they are cut to is not.
    cap_part_ = 0;
    for (auto &L : layers_) cap_part_ = std::max(cap_part_, plan_wgrad(L, nmax).most * (L.nw + L.cout));
    ALLOC(d_part_, float, std::max<int64_t>(cap_part_, kColBlocks * 4096));
    {
        const std::vector<PrepArgs> jobs = prep_jobs(layers_, d_params_);
        ALLOC(d_prep_, PrepArgs, jobs.size());
        if (hipMemcpy(d_prep_, jobs.data(), sizeof(PrepArgs) * jobs.size(), hipMemcpyHostToDevice) != hipSuccess)
            return {HIP_ERROR, "weight-layout table upload failed"};
        n_prep_ = (int32_t)jobs.size();
        max_prep_ = 0;
        for (const auto &j : jobs) max_prep_ = std::max<int64_t>(max_prep_, (int64_t)j.nph * j.npad * j.taps * j.crow);
    }
#undef ALLOC
    if (sizeof(float) * nparam_ >= HostCopy::kLeast) host_copy_.create();

    // He-normal weights, zero biases, zero optimiser state
    for (auto &L : layers_) {
        const float sd = (float)std::sqrt(2.0 / ((double)taps_of(L.kind) * L.cin));
        hipLaunchKernelGGL(init_normal_kernel, dim3(nblk(L.nw)), dim3(256), 0, s, d_params_ + L.w_off, L.nw, sd, seed,
                           L.w_off);
        hipLaunchKernelGGL(fill_f32_kernel, dim3(nblk(L.cout)), dim3(256), 0, s, d_params_ + L.b_off,
                           (int64_t)L.cout, 0.0f);
    }
    hipLaunchKernelGGL(fill_f32_kernel, dim3(nblk(nparam_)), dim3(256), 0, s, d_m_, nparam_, 0.0f);
    hipLaunchKernelGGL(fill_f32_kernel, dim3(nblk(nparam_)), dim3(256), 0, s, d_v_, nparam_, 0.0f);
    hipLaunchKernelGGL(fill_f32_kernel, dim3(nblk(nparam_)), dim3(256), 0, s, d_grads_, nparam_, 0.0f);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = prep_weights(s);
    if (e != hipSuccess) return {HIP_ERROR, hipGetErrorString(e)};
    return {OK, ""};
}

void Net::destroy()
{
    for (void *p : allocs_) (void)hipFree(p);
    allocs_.clear();
    layers_.clear();
}

hipError_t Net::prep_weights(hipStream_t s)
{
    if (n_prep_ == 0) return hipSuccess;
    const int64_t gx = std::min<int64_t>(nblk(max_prep_), 1024);
    hipLaunchKernelGGL(prep_weights_kernel, dim3((unsigned)gx, (unsigned)n_prep_), dim3(256), 0, s,
                       (const PrepArgs *)d_prep_);
    return hipGetLastError();
}

template <int K, int D>
static void launch_between(const ConvArgs &a, hipStream_t s)
{
    const uint32_t tiles = ((uint32_t)a.batch * a.mz * a.my * a.mx + 31) / 32, cols = a.npad / 32;
    // Two column tiles per wave where that leaves a wave per SIMD (rows read
    // once for both: 39 against 55 us for 131072 rows of 32 -> 64 channels; one
    // tile with fewer: 7.2 against 8.2 us for 4096 rows of 64 -> 128).
    const int nt = a.npad % 64 == 0 && (int64_t)tiles * (cols / 2) >= 1024 ? 2 : 1;
    // Phases one after the other in a wave as long as there are 4 waves per
    // SIMD: 80 us all 8 in one wave, 95 us one per wave for 131072 rows of
    // 64 -> 32 channels, where 16 against 15 us for an eighth of the rows.
    int32_t phases = a.nph;
    const auto waves = [&] { return (int64_t)tiles * (cols / nt) * (a.nph / phases); };
    while (phases > 1 && waves() < 4096) phases /= 2;
    const bool few = waves() < 4096;   // then one wave per workgroup, spread over the chip
    const int wg = few ? 1 : 4;
    const dim3 grid((tiles + wg - 1) / wg, cols / nt, a.nph / phases);
    if (nt == 2)
        hipLaunchKernelGGL((conv_kernel<2, K, D>), grid, dim3(64 * wg), 0, s, a, phases);
    else
        hipLaunchKernelGGL((conv_kernel<1, K, D>), grid, dim3(64 * wg), 0, s, a, phases);
}

static hipError_t launch_conv(const ConvArgs &a, hipStream_t s)
{
    if (a.k == 3 && a.s_in == 1 && a.pad == 1 && a.nph == 1 && a.s_out == 1 && a.cin % 16 == 0) {
        // Input channels per chunk: 16 on grids of at least 256 bricks of 8^3
        // (enough workgroups to overlap one's loads with another's products),
        // 32 on smaller ones (half the barriers).
        const int64_t yx = (int64_t)a.batch * ((a.my + 7) / 8) * ((a.mx + 7) / 8);
        const bool large = yx * ((a.mz + 7) / 8) >= 256;
        // Column tiles per workgroup: two share a halo, one where two would
        // leave CUs without a workgroup (its weights then come over two CUs'
        // memory paths: 12.4 against 13.6 us for 16^3 and 128 -> 128 channels).
        const bool two = a.npad % 64 == 0 && (large || yx * a.mz * (a.npad / 64) >= 256);
        if (large) {
            if (two) launch_conv3_as<16, 2, true>(a, s);
            else launch_conv3_as<16, 1, true>(a, s);
        } else if (a.cin % 32 == 0) {
            if (two) launch_conv3_as<32, 2, true>(a, s);
            else launch_conv3_as<32, 1, true>(a, s);
        } else {
            if (two) launch_conv3_as<32, 2, false>(a, s);
            else launch_conv3_as<32, 1, false>(a, s);
        }
        return hipGetLastError();
    }
    // Steps ahead D: a divisor of a phase's steps.  K = 2 has 8 per 16
    // channels; K = 1 reads the deeper level, a multiple of 32 channels.
    if (a.cin % (a.k == 2 ? 16 : 32) != 0) return hipErrorInvalidValue;
    if (a.k == 2) launch_between<2, 8>(a, s);
    else if (a.cin % 64 == 0) launch_between<1, 4>(a, s);
    else launch_between<1, 2>(a, s);
    return hipGetLastError();
}

hipError_t Net::conv_fwd(const Layer &L, int32_t n, const View &x, const View &y, float *yf, int32_t yf_cs,
                         hipStream_t s)
{
    ConvArgs a{};
    const int lin = L.level_in, lout = L.level_out;
    a.x = x.p;
    a.x_cs = x.cs;
    a.x_co = x.co;
    a.cin = L.cin_buf;
    a.iz = nz_ >> lin;
    a.iy = ny_ >> lin;
    a.ix = nx_ >> lin;
    a.oz = nz_ >> lout;
    a.oy = ny_ >> lout;
    a.ox = nx_ >> lout;
    a.batch = n;
    if (L.kind == Layer::CONV3) {
        a.mz = a.oz, a.my = a.oy, a.mx = a.ox;
        a.k = 3, a.s_in = 1, a.pad = 1, a.nph = 1, a.s_out = 1;
    } else if (L.kind == Layer::DOWN2) {
        a.mz = a.oz, a.my = a.oy, a.mx = a.ox;
        a.k = 2, a.s_in = 2, a.pad = 0, a.nph = 1, a.s_out = 1;
    } else {
        a.mz = a.iz, a.my = a.iy, a.mx = a.ix;
        a.k = 1, a.s_in = 1, a.pad = 0, a.nph = 8, a.s_out = 2;
    }
    a.w = L.wf;
    a.npad = L.npad_f;
    a.bias = d_params_ + L.b_off;
    a.cout = L.cout;
    a.act = yf ? 0 : 1;
    a.y = yf ? nullptr : y.p;
    a.y_cs = y.cs;
    a.y_co = y.co;
    a.yf = yf;
    a.yf_cs = yf_cs;
    return launch_conv(a, s);
}

hipError_t Net::conv_bwd_data(const Layer &L, int32_t n, const View &dy, const View &slope, const View *add,
                              const View &dx, hipStream_t s)
{
    ConvArgs a{};
    const int lin = L.level_in, lout = L.level_out;
    // the pass reads the output-side gradient and writes the input side
    a.x = dy.p;
    a.x_cs = dy.cs;
    a.x_co = dy.co;
    a.cin = L.cout_buf;
    a.iz = nz_ >> lout;
    a.iy = ny_ >> lout;
    a.ix = nx_ >> lout;
    a.oz = nz_ >> lin;
    a.oy = ny_ >> lin;
    a.ox = nx_ >> lin;
    a.batch = n;
    if (L.kind == Layer::CONV3) {
        a.mz = a.oz, a.my = a.oy, a.mx = a.ox;
        a.k = 3, a.s_in = 1, a.pad = 1, a.nph = 1, a.s_out = 1;
    } else if (L.kind == Layer::DOWN2) {   // dx[2q + e] = dy[q] W[e]^T
        a.mz = a.iz, a.my = a.iy, a.mx = a.ix;
        a.k = 1, a.s_in = 1, a.pad = 0, a.nph = 8, a.s_out = 2;
    } else {                               // dx[q] = sum_e dy[2q + e] W[e]^T
        a.mz = a.oz, a.my = a.oy, a.mx = a.ox;
        a.k = 2, a.s_in = 2, a.pad = 0, a.nph = 1, a.s_out = 1;
    }
    a.w = L.wb;
    a.npad = L.npad_b;
    a.bias = nullptr;
    a.cout = L.cin;
    a.act = 0;
    a.slope = slope.p;
    a.sl_cs = slope.cs;
    a.sl_co = slope.co;
    if (add) {
        a.add = add->p;
        a.ad_cs = add->cs;
        a.ad_co = add->co;
    }
    a.y = dx.p;
    a.y_cs = dx.cs;
    a.y_co = dx.co;
    return launch_conv(a, s);
}

hipError_t Net::conv_wgrad(const Layer &L, int32_t n, const View &x, const View &dy, hipStream_t s)
{
    WgradArgs a{};
    const int lin = L.level_in, lout = L.level_out;
    a.x = x.p;
    a.x_cs = x.cs;
    a.x_co = x.co;
    a.x_c = x.c;
    a.iz = nz_ >> lin;
    a.iy = ny_ >> lin;
    a.ix = nx_ >> lin;
    a.oz = nz_ >> lout;
    a.oy = ny_ >> lout;
    a.ox = nx_ >> lout;
    a.batch = n;
    if (L.kind == Layer::CONV3) {
        a.mz = a.oz, a.my = a.oy, a.mx = a.ox;
        a.k = 3, a.s_in = 1, a.pad = 1, a.nph = 1, a.s_out = 1;
    } else if (L.kind == Layer::DOWN2) {
        a.mz = a.oz, a.my = a.oy, a.mx = a.ox;
        a.k = 2, a.s_in = 2, a.pad = 0, a.nph = 1, a.s_out = 1;
    } else {
        a.mz = a.iz, a.my = a.iy, a.mx = a.ix;
        a.k = 1, a.s_in = 1, a.pad = 0, a.nph = 8, a.s_out = 2;
    }
    a.dy = dy.p;
    a.dy_cs = dy.cs;
    a.dy_co = dy.co;
    a.dy_c = dy.c;
    a.cin = L.cin;
    a.cout = L.cout;
    const int slots = taps_of(L.kind);
    const WgradPlan p = plan_wgrad(L, n);
    if (p.chunks * (L.nw + L.cout) > std::max<int64_t>(cap_part_, kColBlocks * 4096)) return hipErrorInvalidValue;
    a.chunk = p.chunk;
    a.part = d_part_;
    const unsigned ctiles = (unsigned)(((L.cin + 31) / 32) * ((L.cout + 31) / 32));
    if (p.bricks)
        hipLaunchKernelGGL(wgrad3_kernel, dim3((unsigned)p.chunks, ctiles, 1), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(wgrad_kernel, dim3((unsigned)p.chunks, ctiles, (unsigned)slots), dim3(256), 0, s, a);
    if (p.bricks) {   // the 27-tap kernel's chunk rows hold the weight, then the bias partials (b_off = w_off + nw)
        hipLaunchKernelGGL(sum_chunks_kernel, dim3(nblk(L.nw + L.cout, kSumElems)), dim3(256), 0, s,
                           (const float *)d_part_, (int32_t)p.chunks, L.nw + L.cout, d_grads_ + L.w_off);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(sum_chunks_kernel, dim3(nblk(L.nw, kSumElems)), dim3(256), 0, s, (const float *)d_part_,
                       (int32_t)p.chunks, L.nw, d_grads_ + L.w_off);
    // bias gradient: column sums of dy over the output positions
    const int64_t npos = positions(lout, n);
    hipLaunchKernelGGL(colsum_kernel, dim3(kColBlocks), dim3(256), 0, s, (const uint16_t *)dy.p, dy.cs, dy.co, L.cout,
                       (uint32_t)npos, d_part_);
    hipLaunchKernelGGL(sum_chunks_kernel, dim3(nblk(L.cout, kSumElems)), dim3(256), 0, s, (const float *)d_part_,
                       (int32_t)kColBlocks, (int64_t)L.cout, d_grads_ + L.b_off);
    return hipGetLastError();
}

hipError_t Net::forward(int32_t n, const float *d_x, float *d_y, hipStream_t s)
{
    if (n < 1 || n > nmax_ || !d_x || !d_y) return hipErrorInvalidValue;
    n_last_ = n;
    const int Lv = levels_;
    std::vector<int32_t> ch(Lv);
    for (int l = 0; l < Lv; ++l) ch[l] = base_ << l;
    const int64_t P0 = positions(0, n);
    hipLaunchKernelGGL(to_bf16_padded_kernel, dim3(nblk(P0 * (cin_pad_ / 8))), dim3(256), 0, s, d_x, cin_, cin_pad_, P0,
                       d_xin_);
    size_t li = 0;
    View h{d_xin_, cin_pad_, 0, cin_pad_};
    hipError_t e = hipSuccess;
    auto chk = [&](hipError_t r) {
        if (r != hipSuccess && e == hipSuccess) e = r;
    };
    fin_.assign(layers_.size(), View{});
    fout_.assign(layers_.size(), View{});
    auto conv = [&](const View &x, const View &y, float *yf, int32_t yf_cs) {
        fin_[li] = x;
        fout_[li] = y;
        chk(conv_fwd(layers_[li], n, x, y, yf, yf_cs, s));
        ++li;
    };
    for (int l = 0; l < Lv; ++l) {
        const View a{ha_[l], ch[l], 0, ch[l]};
        conv(h, a, nullptr, 0);
        const View bo = l < Lv - 1 ? View{cat_[l], 2 * ch[l], 0, ch[l]} : View{hbot_, ch[l], 0, ch[l]};
        conv(a, bo, nullptr, 0);
        if (l < Lv - 1) {
            const View d{hd_[l + 1], ch[l + 1], 0, ch[l + 1]};
            conv(bo, d, nullptr, 0);
            h = d;
        }
    }
    View top{hbot_, ch[Lv - 1], 0, ch[Lv - 1]};
    for (int l = Lv - 2; l >= 0; --l) {
        const View uin = top;
        const View cat{cat_[l], 2 * ch[l], 0, 2 * ch[l]};
        conv(uin, cat.at(ch[l], ch[l]), nullptr, 0);
        const View qa{hqa_[l], ch[l], 0, ch[l]};
        conv(cat, qa, nullptr, 0);
        const View qb{hqb_[l], ch[l], 0, ch[l]};
        conv(qa, qb, nullptr, 0);
        top = qb;
    }
    conv(top, View{}, d_y, cout_);
    return e;
}

hipError_t Net::backward(const float *d_dy, hipStream_t s, int32_t stop_layer)
{
    const int32_t n = n_last_;
    if (n < 1 || !d_dy) return hipErrorInvalidValue;
    bdy_.assign(layers_.size(), View{});
    bdx_.assign(layers_.size(), View{});
    const int Lv = levels_;
    std::vector<int32_t> ch(Lv);
    for (int l = 0; l < Lv; ++l) ch[l] = base_ << l;
    hipError_t e = hipSuccess;
    auto chk = [&](hipError_t r) {
        if (r != hipSuccess && e == hipSuccess) e = r;
    };
    // parameter-order indices of the layers
    std::vector<size_t> ea(Lv), eb(Lv), dn(Lv), up(Lv), qa(Lv), qb(Lv);
    size_t li = 0;
    for (int l = 0; l < Lv; ++l) {
        ea[l] = li++;
        eb[l] = li++;
        if (l < Lv - 1) dn[l] = li++;
    }
    for (int l = Lv - 2; l >= 0; --l) {
        up[l] = li++;
        qa[l] = li++;
        qb[l] = li++;
    }
    const size_t out = li;

    // a layer is done once its weight gradient and (if any) backward-data
    // pass are enqueued; stop_layer ends the pass there (test hook)
    bool stop = false;
    auto wgrad = [&](size_t li, const View &x, const View &dy) {
        bdy_[li] = dy;
        chk(conv_wgrad(layers_[li], n, x, dy, s));
        if ((int32_t)li == stop_layer && li == ea[0]) stop = true;
    };
    auto bdata = [&](size_t li, const View &dy, const View &slope, const View *add, const View &dx) {
        bdx_[li] = dx;
        chk(conv_bwd_data(layers_[li], n, dy, slope, add, dx, s));
        if ((int32_t)li == stop_layer) stop = true;
    };
    const int64_t P0 = positions(0, n);
    hipLaunchKernelGGL(to_bf16_padded_kernel, dim3(nblk(P0 * (cout_pad_ / 8))), dim3(256), 0, s, d_dy, cout_, cout_pad_,
                       P0, d_gy_);
    const View top = Lv == 1 ? View{hbot_, ch[0], 0, ch[0]} : View{hqb_[0], ch[0], 0, ch[0]};
    const View gy{d_gy_, cout_pad_, 0, cout_pad_};
    wgrad(out, top, gy);
    View g{g1_[0], ch[0], 0, ch[0]};
    bdata(out, gy, top, nullptr, g);
    if (stop) return e;
    for (int l = 0; l < Lv - 1; ++l) {
        const View hqa{hqa_[l], ch[l], 0, ch[l]};
        const View cat{cat_[l], 2 * ch[l], 0, 2 * ch[l]};
        const View uin = l == Lv - 2 ? View{hbot_, ch[l + 1], 0, ch[l + 1]} : View{hqb_[l + 1], ch[l + 1], 0, ch[l + 1]};
        wgrad(qb[l], hqa, g);
        const View g2{g2_[l], ch[l], 0, ch[l]};
        bdata(qb[l], g, hqa, nullptr, g2);
        if (stop) return e;
        wgrad(qa[l], cat, g2);
        const View gc{gcat_[l], 2 * ch[l], 0, 2 * ch[l]};
        bdata(qa[l], g2, cat, nullptr, gc);
        if (stop) return e;
        const View gu = gc.at(ch[l], ch[l]);
        wgrad(up[l], uin, gu);
        const View gn{g1_[l + 1], ch[l + 1], 0, ch[l + 1]};
        bdata(up[l], gu, uin, nullptr, gn);
        if (stop) return e;
        g = gn;
    }
    for (int l = Lv - 1; l >= 0; --l) {
        const View ha{ha_[l], ch[l], 0, ch[l]};
        wgrad(eb[l], ha, g);
        const View ga{g2_[l], ch[l], 0, ch[l]};
        bdata(eb[l], g, ha, nullptr, ga);
        if (stop) return e;
        const View in = l == 0 ? View{d_xin_, cin_pad_, 0, cin_pad_} : View{hd_[l], ch[l], 0, ch[l]};
        wgrad(ea[l], in, ga);
        if (stop) return e;
        if (l > 0) {
            const View gd{g1_[l], ch[l], 0, ch[l]};
            bdata(ea[l], ga, in, nullptr, gd);
            if (stop) return e;
            const View skip{cat_[l - 1], 2 * ch[l - 1], 0, ch[l - 1]};
            wgrad(dn[l - 1], skip, gd);
            const View gskip{gcat_[l - 1], 2 * ch[l - 1], 0, ch[l - 1]};
            const View gp{g1_[l - 1], ch[l - 1], 0, ch[l - 1]};
            bdata(dn[l - 1], gd, skip, &gskip, gp);
            if (stop) return e;
            g = gp;
        }
    }
    return e;
}

Net::Status Net::read(int32_t layer, int32_t which, float *h, int64_t count, hipStream_t s)
{
    if (layer < 0 || layer >= (int32_t)layers_.size() || which < 0 || which > 3 || !h || n_last_ < 1)
        return {BAD_SHAPE, "bad layer, tensor or state"};
    const Layer &L = layers_[layer];
    const std::vector<View> &vs = which == 0 ? fin_ : which == 1 ? fout_ : which == 2 ? bdy_ : bdx_;
    if ((size_t)layer >= vs.size() || !vs[layer].p) return {BAD_SHAPE, "tensor not stored"};
    const View v = vs[layer];
    // input-side tensors (forward input, backward-data result) live at the
    // input level with cin channels, output-side ones at the output level
    const bool in_side = which == 0 || which == 3;
    const int32_t c = in_side ? L.cin : L.cout;
    const int64_t npos = positions(in_side ? L.level_in : L.level_out, n_last_);
    if (c > v.c || count != npos * c) return {BAD_SHAPE, "count does not match the tensor"};
    std::vector<uint16_t> tmp((size_t)(npos * v.cs));
    hipError_t e = hipMemcpyAsync(tmp.data(), v.p, tmp.size() * sizeof(uint16_t), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return {HIP_ERROR, hipGetErrorString(e)};
    for (int64_t p = 0; p < npos; ++p)
        for (int32_t j = 0; j < c; ++j) {
            const uint32_t bits = (uint32_t)tmp[(size_t)(p * v.cs + v.co + j)] << 16;
            float f;
            std::memcpy(&f, &bits, sizeof f);
            h[p * c + j] = f;
        }
    return {OK, ""};
}

hipError_t Net::mse(int32_t n, const float *d_y, const float *d_t, float *d_dy, double *h_loss, hipStream_t s)
{
    if (n < 1 || n > nmax_ || !d_y || !d_t) return hipErrorInvalidValue;
    const int64_t count = positions(0, n) * cout_;
    const int blocks = 1024;
    hipLaunchKernelGGL(mse_kernel, dim3(blocks), dim3(256), 0, s, d_y, d_t, count, d_dy, d_loss_part_);
    hipLaunchKernelGGL(sum_f64_kernel, dim3(1), dim3(256), 0, s, (const double *)d_loss_part_, blocks,
                       d_loss_part_ + 1024);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !h_loss) return e;
    double sum = 0.0;
    e = hipMemcpyAsync(&sum, d_loss_part_ + 1024, sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    *h_loss = sum / (double)count;
    return e;
}

hipError_t Net::adam(float lr, float beta1, float beta2, float eps, int32_t step, hipStream_t s)
{
    if (step < 1) return hipErrorInvalidValue;
    const double c1 = 1.0 - std::pow((double)beta1, step);
    const double c2 = 1.0 - std::pow((double)beta2, step);
    // bias-corrected step size; eps scaled so that the update equals m_hat / (sqrt(v_hat) + eps)
    const float lr_t = (float)(lr * std::sqrt(c2) / c1);
    const float eps_t = (float)(eps * std::sqrt(c2));
    hipLaunchKernelGGL(adam_kernel, dim3(nblk(nparam_)), dim3(256), 0, s, d_params_, (const float *)d_grads_, d_m_,
                       d_v_, nparam_, lr_t, beta1, beta2, eps_t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return prep_weights(s);
}

hipError_t Net::zero_grads(hipStream_t s)
{
    hipLaunchKernelGGL(fill_f32_kernel, dim3(nblk(nparam_)), dim3(256), 0, s, d_grads_, nparam_, 0.0f);
    return hipGetLastError();
}

hipError_t Net::set_params(const float *h, hipStream_t s)
{
    hipError_t e = hipMemcpyAsync(d_params_, h, sizeof(float) * nparam_, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    return prep_weights(s);
}

hipError_t Net::get_params(float *h, hipStream_t s)
{
    return host_copy_.copy(h, d_params_, sizeof(float) * nparam_, s);
}

hipError_t Net::get_grads(float *h, hipStream_t s)
{
    return host_copy_.copy(h, d_grads_, sizeof(float) * nparam_, s);
}

int64_t Net::flops_forward(int32_t n) const
{
    int64_t f = 0;
    for (auto &L : layers_) {
        const int64_t rows = positions(L.level_out, n);   // an up convolution: 8 phases x coarse rows
        const int64_t k = L.kind == Layer::CONV3 ? 27 * (int64_t)L.cin : L.kind == Layer::DOWN2 ? 8 * (int64_t)L.cin
                                                                                                 : (int64_t)L.cin;
        f += 2 * rows * k * L.cout;
    }
    return f;
}

}  // namespace unet
}  // namespace soc
