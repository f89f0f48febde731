// msz_net.hip -- the learned edit proposal: a 3-layer 3x3x3 conv net whose
// prediction warm-starts the correction loop (the loop still runs after it
// and judges).  BF16 weights and activations, FP32 accumulation, on MFMA.
//
// Parameters (FP32 master copy, one flat array, MSZ_NET_PARAMS floats):
//   W0[27][16][16] b0[16]      features (12 used, 16 stored) -> 16
//   W1[27][16][16] b1[16]      16 -> 16
//   W2[27][16]     b2[1]       16 -> 1
// tap = (dz+1)*9 + (dy+1)*3 + (dx+1); zero padding outside the grid.
// Activations: BF16, channel-last [vertex][16], vertex id x + nx*(y + ny*z).
//
// Convolution as GEMM on v_mfma_f32_16x16x32_bf16: M = 16 output channels,
// N = 16 x-consecutive vertices, K = 32 (tap, input channel) pairs per
// instruction.  A (weights) stays in registers for the whole kernel, B is a
// 16-byte read of 8 consecutive channels of one shifted vertex from the LDS
// input tile; a lane's result is 4 consecutive output channels of one vertex,
// written as one 8-byte store.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "msz_internal.h"

namespace msz {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kOffW0 = 0, kOffB0 = kOffW0 + 27 * 16 * 16, kOffW1 = kOffB0 + 16, kOffB1 = kOffW1 + 27 * 16 * 16,
              kOffW2 = kOffB1 + 16, kOffB2 = kOffW2 + 27 * 16, kNetParams = kOffB2 + 1;
static_assert(kNetParams == MSZ_NET_PARAMS, "parameter layout");

// Conv tile: 16 (x) x TY x TZ output vertices, 256 threads = 4 waves.
template <int TY, int TZ>
struct ConvTile {
    static constexpr int X = 16, Y = TY, Z = TZ, HX = X + 2, HY = Y + 2, HZ = Z + 2;
    static constexpr int HALO = HX * HY * HZ;
    static constexpr int ROWS = Y * Z;  // x-rows of 16 vertices
};

__device__ __forceinline__ uint16_t bf16_bits(float v) {
    const __bf16 b = static_cast<__bf16>(v);  // round to nearest even
    return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float bf16_float(uint16_t u) { return __uint_as_float(static_cast<unsigned>(u) << 16); }

__device__ __forceinline__ void tap_delta(int tap, int& dx, int& dy, int& dz) {
    dz = tap / 9 - 1;
    dy = (tap / 3) % 3 - 1;
    dx = tap % 3 - 1;
}

// Weight source of one convolution launch: value(tap, in, out) =
//   W[(flip ? 26 - tap : tap) * s_tap + in * s_in + out * s_out]
// for in < n_in and out < n_out, zero otherwise (padding channels and taps).
struct WeightView {
    const float* W;
    const float* bias;  // n_out entries or nullptr
    int s_tap, s_in, s_out, n_in, n_out, flip;
};

__device__ __forceinline__ float weight_at(const WeightView& wv, int tap, int in, int out) {
    if (tap >= 27 || in >= wv.n_in || out >= wv.n_out) return 0.0f;
    const int t = wv.flip ? 26 - tap : tap;
    return wv.W[t * wv.s_tap + in * wv.s_in + out * wv.s_out];
}

// Input tile t of a convolution: 16 x TY x TZ vertices plus a one-vertex halo,
// two 16-byte chunks (eight channels each) per vertex, zeros outside the grid.
// Chunk e of the tile is chunk e % 2 of halo vertex e / 2.
struct TileOrigin {
    int X0, Y0, Z0;
};
template <int TY, int TZ>
__device__ __forceinline__ TileOrigin conv_origin(int t, int tx_n, int ty_n) {
    using T = ConvTile<TY, TZ>;
    return {(t % tx_n) * T::X, ((t / tx_n) % ty_n) * T::Y, (t / (tx_n * ty_n)) * T::Z};
}

template <int TY, int TZ>
__device__ __forceinline__ uint4 conv_chunk(const uint16_t* __restrict__ in, const Grid& gr, const TileOrigin& o,
                                            int e) {
    using T = ConvTile<TY, TZ>;
    const int hv = e >> 1, ch = e & 1;
    const int hx = hv % T::HX, hy = (hv / T::HX) % T::HY, hz = hv / (T::HX * T::HY);
    const int x = o.X0 + hx - 1, y = o.Y0 + hy - 1, z = o.Z0 + hz - 1;
    // an unconditional load (vertex 0 outside the grid), so that a thread's
    // loads are all issued before the first one is waited for
    const bool ok = x >= 0 && x < gr.nx && y >= 0 && y < gr.ny && z >= 0 && z < gr.nz;
    const long vid = ok ? x + static_cast<long>(gr.nx) * y + static_cast<long>(gr.nxy) * z : 0;
    const uint4 v = reinterpret_cast<const uint4*>(in)[2 * vid + ch];
    return make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
}

template <int TY, int TZ, int PER>
__device__ __forceinline__ void conv_tile_load(const uint16_t* __restrict__ in, const Grid& gr, int t, int tx_n,
                                               int ty_n, uint4 (&buf)[PER]) {
    const TileOrigin o = conv_origin<TY, TZ>(t, tx_n, ty_n);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = threadIdx.x + 256 * k;
        buf[k] = conv_chunk<TY, TZ>(in, gr, o, min(e, 2 * ConvTile<TY, TZ>::HALO - 1));
    }
}

enum : int { kConvHidden = 0, kConvBackData = 1 };

// out = conv(in) for 16 input and 16 output channels.
//  kConvHidden:   out16[v][16] = bf16(relu(conv + bias))
//  kConvBackData: out16[v][16] = bf16(conv * (mask[v][c] > 0))  (gradient through ReLU)
//
// A row of 16 vertices takes 14 MFMAs in one chain, each with one 16-byte LDS
// read per lane.  Four y-consecutive rows run side by side, so the chains
// overlap, and a lane's LDS offset is one of 14 registers plus a row constant.
// Bound by the LDS reads (8 cycles of the compute unit per MFMA, which takes
// 4) and the 64 bytes per vertex it moves, about 210 us each for 256^3: 338 us
// there, where one chain at a time with its address arithmetic took 468; for
// 128^3, where loading the weights weighed more, 54 against 139.
template <int TY, int TZ, int MODE>
__global__ void __launch_bounds__(256) k_conv(const uint16_t* __restrict__ in, Grid gr, WeightView wv,
                                              const uint16_t* __restrict__ mask, uint16_t* __restrict__ out16) {
    using T = ConvTile<TY, TZ>;
    constexpr int KSTEPS = 14;  // 27 taps and one zero tap, two per MFMA
    constexpr int R = 4;        // rows computed side by side
    static_assert(T::Y % R == 0 && T::ROWS % (4 * R) == 0, "whole row groups per wave");
    __shared__ uint4 tile[T::HALO * 2];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, g = lane >> 4;

    // the weights as BF16 [out][tap][in] in the tile's LDS first: one strided
    // global load per thread and tap, where a lane picking its own 112 values
    // from memory cost each block some 35 us
    static_assert(16 * 28 * 2 <= T::HALO * 2, "the weights fit the tile's LDS");
    uint16_t* wl = reinterpret_cast<uint16_t*>(tile);
#pragma unroll
    for (int tap = 0; tap < 28; ++tap) {
        const int ci = threadIdx.x >> 4, co = threadIdx.x & 15;
        wl[(co * 28 + tap) * 16 + ci] = bf16_bits(weight_at(wv, tap, ci, co));
    }
    __syncthreads();

    // A operand (weights) and the lane's tile offset (in chunks) of every K
    // step, in registers for the whole kernel
    bf16x8 wa[KSTEPS];
    int off[KSTEPS];
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) {
        const int tap = 2 * s + (g >> 1);
        wa[s] = __builtin_bit_cast(bf16x8, tile[(m * 28 + tap) * 2 + (g & 1)]);
        int dx, dy, dz;
        tap_delta(tap > 26 ? 26 : tap, dx, dy, dz);  // the zero-weight padding tap reads a valid address
        off[s] = 2 * ((m + dx + 1) + T::HX * ((dy + 1) + T::HY * (dz + 1))) + (g & 1);
    }
    float bias[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int co = 4 * g + i;
        bias[i] = (wv.bias && co < wv.n_out) ? wv.bias[co] : 0.0f;
    }

    const int tx_n = (gr.nx + T::X - 1) / T::X, ty_n = (gr.ny + T::Y - 1) / T::Y, tz_n = (gr.nz + T::Z - 1) / T::Z;
    const int ntiles = tx_n * ty_n * tz_n;
    const ItemRange range = xcd_items(ntiles);
    // the input tile (with halo) of the next tile is loaded into registers
    // while the current one is computed from LDS
    constexpr int NCH = T::HALO * 2;
    constexpr int PER = (NCH + 255) / 256;
    uint4 buf[PER];
    if (range.first < range.hi) conv_tile_load<TY, TZ, PER>(in, gr, range.first, tx_n, ty_n, buf);
    for (int t = range.first; t < range.hi; t += range.stride) {
        const TileOrigin o = conv_origin<TY, TZ>(t, tx_n, ty_n);
        __syncthreads();  // the previous tile's reads are done
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = threadIdx.x + 256 * k;
            if (e < NCH) tile[e] = buf[k];
        }
        __syncthreads();
        if (t + range.stride < range.hi) conv_tile_load<TY, TZ, PER>(in, gr, t + range.stride, tx_n, ty_n, buf);

#pragma unroll 1
        for (int q = 0; q < T::ROWS / (4 * R); ++q) {
            const int row = wave * (T::ROWS / 4) + q * R;  // the first of R rows
            const int ly = row % T::Y, lz = row / T::Y;
            const uint4* src = tile + 2 * T::HX * (ly + T::HY * lz);
            f32x4 acc[R];
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s) {
                const uint4* b = src + off[s];
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        wa[s], __builtin_bit_cast(bf16x8, b[2 * T::HX * r]), acc[r], 0, 0, 0);
            }
            const int x = o.X0 + m, z = o.Z0 + lz;
            if (x >= gr.nx || z >= gr.nz) continue;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int y = o.Y0 + ly + r;
                if (y >= gr.ny) break;
                const long vid = x + static_cast<long>(gr.nx) * y + static_cast<long>(gr.nxy) * z;
                uint16_t ov[4];
                if constexpr (MODE == kConvHidden) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) ov[i] = bf16_bits(fmaxf(acc[r][i] + bias[i], 0.0f));
                } else {
                    const uint2 mk = reinterpret_cast<const uint2*>(mask)[vid * 4 + g];
                    const uint16_t mv[4] = {static_cast<uint16_t>(mk.x & 0xFFFFu), static_cast<uint16_t>(mk.x >> 16),
                                            static_cast<uint16_t>(mk.y & 0xFFFFu), static_cast<uint16_t>(mk.y >> 16)};
#pragma unroll
                    for (int i = 0; i < 4; ++i) ov[i] = bf16_float(mv[i]) > 0.0f ? bf16_bits(acc[r][i]) : 0;
                }
                uint2 pk;
                pk.x = static_cast<unsigned>(ov[0]) | (static_cast<unsigned>(ov[1]) << 16);
                pk.y = static_cast<unsigned>(ov[2]) | (static_cast<unsigned>(ov[3]) << 16);
                reinterpret_cast<uint2*>(out16)[vid * 4 + g] = pk;
            }
        }
    }
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// The output layer (16 -> 1 channels) with packed BF16 dot products on the
// VALU (v_dot2 accumulates two products into an FP32 sum): on the 16x16 MFMA
// tile it would use one of 16 output rows.  A thread computes OPT
// y-consecutive outputs of one x, so the 16 lanes of a row read 16
// consecutive vertices; the two chunks of a vertex lie in two LDS arrays,
// which makes such a read contiguous (threads that owned x-consecutive
// outputs read 128 bytes apart, and bank conflicts bound the kernel:
// 256^3 took 713 us and takes 285).  An output adds its taps in increasing order.
template <int TY, int TZ>
__global__ void __launch_bounds__(256) k_conv_out(const uint16_t* __restrict__ in, Grid gr,
                                                  const float* __restrict__ W2, const float* __restrict__ b2,
                                                  float* __restrict__ out1) {
    using T = ConvTile<TY, TZ>;
    constexpr int OPT = 16 * T::ROWS / 256;  // outputs per thread: 4 for 8 x 8 rows, 2 for 32 x 1
    static_assert(OPT * 256 == 16 * T::ROWS && T::Y % OPT == 0, "every output has one thread");
    __shared__ uint4 tile[2][T::HALO];
    __shared__ uint4 wq[27 * 2];  // BF16 weights of every tap, channels 0..7 and 8..15
    for (int e = threadIdx.x; e < 27 * 8; e += 256)
        reinterpret_cast<unsigned*>(wq)[e] = static_cast<unsigned>(bf16_bits(W2[2 * e])) |
                                             (static_cast<unsigned>(bf16_bits(W2[2 * e + 1])) << 16);
    const float bias = b2[0];
    const int lx = threadIdx.x & 15, ly = OPT * ((threadIdx.x >> 4) % (T::Y / OPT)),
              lz = (threadIdx.x >> 4) / (T::Y / OPT);

    const int tx_n = (gr.nx + T::X - 1) / T::X, ty_n = (gr.ny + T::Y - 1) / T::Y, tz_n = (gr.nz + T::Z - 1) / T::Z;
    const ItemRange range = xcd_items(tx_n * ty_n * tz_n);
    constexpr int NCH = T::HALO * 2;
    constexpr int PER = (NCH + 255) / 256;
    uint4 buf[PER];
    if (range.first < range.hi) conv_tile_load<TY, TZ, PER>(in, gr, range.first, tx_n, ty_n, buf);
    for (int t = range.first; t < range.hi; t += range.stride) {
        const TileOrigin o = conv_origin<TY, TZ>(t, tx_n, ty_n);
        __syncthreads();  // the previous tile's reads (and the weight packing) are done
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = threadIdx.x + 256 * k;
            if (e < NCH) tile[e & 1][e >> 1] = buf[k];
        }
        __syncthreads();
        if (t + range.stride < range.hi) conv_tile_load<TY, TZ, PER>(in, gr, t + range.stride, tx_n, ty_n, buf);
        float acc[OPT];
#pragma unroll
        for (int i = 0; i < OPT; ++i) acc[i] = bias;
#pragma unroll 1
        for (int dz = 0; dz < 3; ++dz) {
            unsigned w[9][8];  // the plane's nine taps
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const uint4 a = wq[18 * dz + 2 * k], b = wq[18 * dz + 2 * k + 1];
                w[k][0] = a.x, w[k][1] = a.y, w[k][2] = a.z, w[k][3] = a.w;
                w[k][4] = b.x, w[k][5] = b.y, w[k][6] = b.z, w[k][7] = b.w;
            }
            // input row r is the row dy = r - i (0..2) of output i
#pragma unroll
            for (int r = 0; r < OPT + 2; ++r)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    const int hv = lx + dx + T::HX * (ly + r + T::HY * (lz + dz));
                    const uint4 u0 = tile[0][hv], u1 = tile[1][hv];
                    const unsigned col[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
#pragma unroll
                    for (int i = 0; i < OPT; ++i) {
                        const int dy = r - i;
                        if (dy < 0 || dy > 2) continue;
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            acc[i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, col[q]),
                                                                     __builtin_bit_cast(bf16x2, w[3 * dy + dx][q]),
                                                                     acc[i], false);
                    }
                }
        }
        const int x = o.X0 + lx, z = o.Z0 + lz;
        if (x < gr.nx && z < gr.nz) {
#pragma unroll
            for (int i = 0; i < OPT; ++i) {
                const int y = o.Y0 + ly + i;
                if (y < gr.ny) out1[x + static_cast<long>(gr.nx) * y + static_cast<long>(gr.nxy) * z] = acc[i];
            }
        }
    }
}

// Weight gradient of one layer, one partial sum per block:
//   part[block][tap][ci][co]     = sum over the block's vertices v of in[v + tap][ci] * dz[v][co]
//   part[block][27 * 256 + co]   = sum over the block's vertices v of dz[v][co]
// M = 16 input channels, N = 16 output channels, K = 32 vertices (two rows of
// 16) per MFMA.  Both operands need eight vertices of one channel per lane,
// while a vertex's channels are contiguous: ds_read_b64_tr_b16 hands each of
// 16 lanes its channel of four consecutive vertices (128 contiguous bytes),
// for any tap at a constant offset from the lane's address, so the inner loop
// is two LDS reads and one MFMA per tap.  A wave keeps the sums of all 27
// taps (and of dz, against a row of ones) in registers over all tiles of its
// block; the waves' sums are added at the end.  Bound by the LDS reads (8
// cycles of the compute unit per MFMA) and the staging of the tiles:
// 128^3 takes 61 us where one pass per tap with 2-byte reads took 464.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kDwSums = 27 * 256 + 16;  // sums of one partial
constexpr int kDwBlocks = 768;          // three per compute unit (51 KB of LDS each)

// Eight vertices of the lane's channel: the four at p (a group of 16 lanes
// passes 128 contiguous bytes, 8 per lane) and the four after them.
__device__ __forceinline__ bf16x8 read_vertices8(const uint16_t* p) {
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 64));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int TY, int TZ>
__global__ void __launch_bounds__(256, 3) k_conv_dw(const uint16_t* __restrict__ in, const uint16_t* __restrict__ dz,
                                                 Grid gr, float* __restrict__ part) {
    using T = ConvTile<TY, TZ>;
    constexpr int NV = T::X * T::ROWS;
    static_assert(T::Y % 2 == 0 && T::ROWS % 8 == 0, "row pairs split evenly over four waves");
    union Smem {
        uint4 stage[T::HALO * 2 + NV * 2];
        float sums[kDwSums];
    };
    __shared__ Smem sm;
    uint4* sin = sm.stage;
    uint4* sdz = sm.stage + T::HALO * 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int tx_n = (gr.nx + T::X - 1) / T::X, ty_n = (gr.ny + T::Y - 1) / T::Y, tz_n = (gr.nz + T::Z - 1) / T::Z;
    const ItemRange range = xcd_items(tx_n * ty_n * tz_n);
    f32x4 acc[27], acc_b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tap = 0; tap < 27; ++tap) acc[tap] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = static_cast<__bf16>(1.0f);
    for (int t = range.first; t < range.hi; t += range.stride) {
        const TileOrigin o = conv_origin<TY, TZ>(t, tx_n, ty_n);
        __syncthreads();  // the previous tile's reads are done
        // in two batches of loads (the sums leave few registers)
        constexpr int NCH = T::HALO * 2, PER = (NCH + 255) / 256, HALF = (PER + 1) / 2;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint4 buf[HALF];
#pragma unroll
            for (int k = 0; k < HALF; ++k)
                if (h * HALF + k < PER)
                    buf[k] = conv_chunk<TY, TZ>(in, gr, o, min(static_cast<int>(threadIdx.x) + 256 * (h * HALF + k), NCH - 1));
#pragma unroll
            for (int k = 0; k < HALF; ++k) {
                const int e = threadIdx.x + 256 * (h * HALF + k);
                if (h * HALF + k < PER && e < NCH) sin[e] = buf[k];
            }
        }
        uint4 db[NV * 2 / 256];
#pragma unroll
        for (int k = 0; k < NV * 2 / 256; ++k) {
            const int e = threadIdx.x + 256 * k, lv = e >> 1, r = lv / T::X;
            const int x = o.X0 + lv % T::X, y = o.Y0 + r % T::Y, z = o.Z0 + r / T::Y;
            const bool ok = x < gr.nx && y < gr.ny && z < gr.nz;  // the others contribute nothing
            const uint4 v = reinterpret_cast<const uint4*>(
                dz)[ok ? 2 * (x + static_cast<long>(gr.nx) * y + static_cast<long>(gr.nxy) * z) + (e & 1) : 0];
            db[k] = make_uint4(ok ? v.x : 0u, ok ? v.y : 0u, ok ? v.z : 0u, ok ? v.w : 0u);
        }
#pragma unroll
        for (int k = 0; k < NV * 2 / 256; ++k) sdz[threadIdx.x + 256 * k] = db[k];
        __syncthreads();
#pragma unroll 1
        for (int q = wave; q < T::ROWS / 2; q += 4) {
            // lanes 16 g ..: vertices 8 (g & 1) .. + 7 of row 2 q + (g >> 1)
            const int row = 2 * q + (g >> 1), x = 8 * (g & 1), ly = row % T::Y, lz = row / T::Y;
            const uint16_t* pd = reinterpret_cast<const uint16_t*>(sdz) + 16 * (x + T::X * row) + 4 * m;
            // the lane's vertices displaced by tap (-1, -1, -1)
            const uint16_t* pi = reinterpret_cast<const uint16_t*>(sin) + 16 * (x + T::HX * (ly + T::HY * lz)) + 4 * m;
            const bf16x8 b = read_vertices8(pd);
#pragma unroll
            for (int tap = 0; tap < 27; ++tap) {
                int dx, dy, dzz;
                tap_delta(tap, dx, dy, dzz);
                const bf16x8 a = read_vertices8(pi + 16 * ((dx + 1) + T::HX * ((dy + 1) + T::HY * (dzz + 1))));
                acc[tap] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[tap], 0, 0, 0);
            }
            acc_b = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, b, acc_b, 0, 0, 0);
        }
    }
    // acc[tap][i] = D[ci = 4g + i][co = m]; the waves in turn
    for (int w = 0; w < 4; ++w) {
        __syncthreads();
        if (wave != w) continue;
#pragma unroll
        for (int tap = 0; tap < 27; ++tap)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float* d = sm.sums + tap * 256 + (4 * g + i) * 16 + m;
                *d = w == 0 ? acc[tap][i] : *d + acc[tap][i];
            }
        if (g == 0) {  // every row of acc_b is the sum of dz
            float* d = sm.sums + 27 * 256 + m;
            *d = w == 0 ? acc_b[0] : *d + acc_b[0];
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kDwSums; e += 256) part[static_cast<long>(blockIdx.x) * kDwSums + e] = sm.sums[e];
}

// Sums the blocks' partials into the gradient of one layer's weights and bias,
// in the parameter layout (out channels beyond n_out are dropped).  A block
// sums 64 entries: its 16 waves take every 16th partial each, so that one
// entry is not a serial chain of loads over all partials (6 us for 768
// partials; one thread per entry over 2048 partials took 480).
__global__ void __launch_bounds__(1024) k_reduce_dw(const float* __restrict__ part, int nparts, int n_out,
                                                    float* __restrict__ gW, float* __restrict__ gb) {
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, seg = threadIdx.x >> 6, e = blockIdx.x * 64 + lane;
    float s = 0.0f;
    if (e < kDwSums) {
#pragma unroll 8
        for (int b = seg; b < nparts; b += 16) s += part[static_cast<long>(b) * kDwSums + e];
    }
    red[seg][lane] = s;
    __syncthreads();
    if (seg != 0 || e >= kDwSums) return;
    for (int k = 1; k < 16; ++k) s += red[k][lane];
    if (e < 27 * 256) {
        const int co = e % 16;
        if (co < n_out) gW[(e / 16) * n_out + co] = s;
    } else if (e - 27 * 256 < n_out) {
        gb[e - 27 * 256] = s;
    }
}

// Input channels of the net (16 stored per vertex, 12 used; the box is the
// 3x3x3 block around the vertex clipped to the grid, the clamps are [-8, 8]):
//   0 (fhat - box mean of fhat) / xi     1 log10(xi / value range) / 4 + 1
//   2..5 FPmax, FPmin, FNmax, FNmin of fhat against f
//   6 (fhat - f) / xi                    7 (f - box mean of f) / xi
//   8 dn_f(u) = i for an FPmin neighbour u       9 up_fhat(u) = i for an FNmax neighbour u
//   10 dn_f(u) = i for a neighbour u with dn_fhat(u) != dn_f(u)
//   11 up_fhat(u) = i for a neighbour u with up_fhat(u) != up_f(u)
// Channels 8..11 gather over the neighbour slots: neighbour j = i + off[s]
// points back at i through the opposite slot s ^ 1.
//
// A block owns FX x FY columns and walks kFeatZ planes of z.  Each plane, with
// a one-vertex halo, is staged in LDS once: (f, fhat) and the target masks of
// every vertex, both zero outside the grid (a zero adds nothing to a box sum
// and targets nothing).  A thread reads its 3 x 3 neighbourhood and carries
// what the planes above and below need of it in registers: the box sums of
// planes z - 1 and z, and the target bits it hands to each side.  Quotients
// by the box count and by xi are correctly rounded, as the division is (the
// reciprocals are correctly rounded and no divisor's significand is all ones).
// Moves 42 bytes per vertex: 213 us for 256^3 (3.3 TB/s), where one thread
// per column, loading its 36 values per vertex itself, took 788.
constexpr int kFeatZ = 16;
template <int FX, int FY>
struct FeatTile {
    static constexpr int X = FX, Y = FY, HX = FX + 2, HY = FY + 2;
    static_assert(FX * FY == 256, "a thread per column");
};

// Target masks of vertex j from its directions in f and fhat: bit d of a is
// set when j's descents differ and f's is slot d, bit d of b when its ascents
// differ and fhat's is slot d (bit 15: the self slot); the high halves repeat
// a where fhat's descent is the self slot and b where f's ascent is.
struct TargetMask {
    unsigned a, b;
};
__device__ __forceinline__ TargetMask target_mask(unsigned fj, unsigned hj) {
    const unsigned uf = fj >> 4, nf = fj & 15u, uh = hj >> 4, nh = hj & 15u;
    const unsigned a = nh != nf ? 1u << nf : 0u, b = uh != uf ? 1u << uh : 0u;
    return {nh == kSelf ? a | (a << 16) : a, uf == kSelf ? b | (b << 16) : b};
}

// Bits 0 and 16 of each word: the vertex with mask w, in slot s of the
// reader, targets the reader.
__device__ __forceinline__ void add_target(uint2& t, const uint2& w, int s) {
    t.x |= (w.x >> (s ^ 1)) & 0x00010001u;
    t.y |= (w.y >> (s ^ 1)) & 0x00010001u;
}

// x / d for a positive finite d, r = 1 / d: a reciprocal, one residual and one
// correction (Markstein's method), and the product itself where that is a zero
// or an infinity (the residual would lose the sign of the one and make the
// other not a number; no other product is either, x being a sum of a few
// float32 values).
__device__ __forceinline__ double quotient(double x, double d, double r) {
    const double q = __dmul_rn(x, r);
    return q + q == q ? q : __fma_rn(__fma_rn(-q, d, x), r, q);
}

template <int FX, int FY>
__global__ void __launch_bounds__(256) k_features(const float* __restrict__ f, const float* __restrict__ fhat,
                                                  const uint8_t* __restrict__ dirs_f,
                                                  const uint8_t* __restrict__ dirs_h, Grid gr, int ntiles, float xi,
                                                  float xi_ch, uint16_t* __restrict__ feat) {
    using T = FeatTile<FX, FY>;
    constexpr int NP = T::HX * T::HY, PER = (NP + 255) / 256;
    __shared__ float2 sv[2][NP];
    __shared__ uint2 st[2][NP];
    const int tx_n = (gr.nx + T::X - 1) / T::X, ty_n = (gr.ny + T::Y - 1) / T::Y;
    const int t = blockIdx.y * gridDim.x + blockIdx.x;
    if (t >= ntiles) return;
    const int X0 = (t % tx_n) * T::X, Y0 = ((t / tx_n) % ty_n) * T::Y, Z0 = (t / (tx_n * ty_n)) * kFeatZ;
    const int lx = threadIdx.x % T::X, ly = threadIdx.x / T::X;
    const int x = X0 + lx, y = Y0 + ly;
    const bool in_xy = x < gr.nx && y < gr.ny;
    const int z_end = min(Z0 + kFeatZ, gr.nz);  // planes [Z0, z_end) are written
    const int n_xy = (1 + (x > 0) + (x + 1 < gr.nx)) * (1 + (y > 0) + (y + 1 < gr.ny));
    const double xid = xi, rxi = 1.0 / xid;
    const unsigned one = bf16_bits(1.0f);

    // plane z into registers (unconditional loads; zeros outside the grid,
    // two planes of the three of a 2D field)
    float2 rv[PER];
    uint2 rt[PER];
    auto load = [&](int z) {
        if (z < 0 || z >= gr.nz) {
#pragma unroll
            for (int k = 0; k < PER; ++k) rv[k] = make_float2(0.0f, 0.0f), rt[k] = make_uint2(0u, 0u);
            return;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = min(static_cast<int>(threadIdx.x) + 256 * k, NP - 1);
            const int xx = X0 + e % T::HX - 1, yy = Y0 + e / T::HX - 1;
            const bool ok = xx >= 0 && xx < gr.nx && yy >= 0 && yy < gr.ny;
            const long j = ok ? xx + static_cast<long>(gr.nx) * yy + static_cast<long>(gr.nxy) * z : 0;
            const float fj = f[j], hj = fhat[j];
            const TargetMask m = target_mask(dirs_f[j], dirs_h[j]);
            rv[k] = make_float2(ok ? fj : 0.0f, ok ? hj : 0.0f);
            rt[k] = make_uint2(ok ? m.a : 0u, ok ? m.b : 0u);
        }
    };
    auto store = [&](int slot) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = threadIdx.x + 256 * k;
            if (e < NP) sv[slot][e] = rv[k], st[slot][e] = rt[k];
        }
    };

    // carried from plane to plane: box sums of the last two planes, the last
    // plane's target bits within itself and those of the two planes before,
    // the vertex's values
    double sf_m = 0.0, sh_m = 0.0, sf_0 = 0.0, sh_0 = 0.0;
    uint2 t_0 = make_uint2(0u, 0u), t_dn = t_0, t_hold = t_0, m_0 = t_0;
    float2 v_0 = make_float2(0.0f, 0.0f);
    int n_last = 0;
    double r_last = 0.0;

    load(Z0 - 1);
    store(0);
    __syncthreads();
    for (int z = Z0 - 1; z <= z_end; ++z) {  // plane z is in LDS; vertex z - 1 is written
        const int slot = (z - Z0 + 1) & 1;
        if (z < z_end) load(z + 1);
        const float2* pv = sv[slot] + (lx + 1) + T::HX * (ly + 1);
        const uint2* pt = st[slot] + (lx + 1) + T::HX * (ly + 1);
        double sf = 0.0, sh = 0.0;
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
            for (int dx = -1; dx <= 1; ++dx) {
                const float2 v = pv[dx + T::HX * dy];
                sf += v.x;
                sh += v.y;
            }
        const uint2 c = pt[0], px = pt[1], mx = pt[-1], py = pt[T::HX], my = pt[-T::HX], pxy = pt[T::HX + 1],
                    mxy = pt[-T::HX - 1];
        uint2 t_up = make_uint2(0u, 0u), t_in = t_up, t_next = t_up;
        add_target(t_up, c, 6);  // this plane's vertices seen from the plane below it
        add_target(t_up, px, 8);
        add_target(t_up, py, 10);
        add_target(t_up, pxy, 12);
        add_target(t_in, px, 0);
        add_target(t_in, mx, 1);
        add_target(t_in, py, 2);
        add_target(t_in, my, 3);
        add_target(t_in, pxy, 4);
        add_target(t_in, mxy, 5);
        add_target(t_next, c, 7);  // and from the plane above it
        add_target(t_next, mx, 9);
        add_target(t_next, my, 11);
        add_target(t_next, mxy, 13);
        if (z > Z0 && in_xy) {
            const int zc = z - 1;
            const int n = n_xy * (1 + (zc > 0) + (zc + 1 < gr.nz));
            if (n != n_last) n_last = n, r_last = 1.0 / n;
            const double hi = v_0.y, fi = v_0.x;
            const double bh = quotient(sh_m + sh_0 + sh, n, r_last), bf = quotient(sf_m + sf_0 + sf, n, r_last);
            const float ch0 = fminf(fmaxf(static_cast<float>(quotient(hi - bh, xid, rxi)), -8.0f), 8.0f);
            const float ch6 = fminf(fmaxf(static_cast<float>(quotient(hi - fi, xid, rxi)), -8.0f), 8.0f);
            const float ch7 = fminf(fmaxf(static_cast<float>(quotient(fi - bf, xid, rxi)), -8.0f), 8.0f);
            const unsigned ta = t_0.x | t_up.x | t_dn.x, tb = t_0.y | t_up.y | t_dn.y;
            uint4 o0, o1;
            o0.x = static_cast<unsigned>(bf16_bits(ch0)) | (static_cast<unsigned>(bf16_bits(xi_ch)) << 16);
            // the vertex's own cases: its ascents differ and fhat's is itself (FPmax), ...
            o0.y = ((m_0.y & 0x8000u) ? one : 0u) | ((m_0.x >> 16) ? one << 16 : 0u);
            o0.z = ((m_0.y >> 16) ? one : 0u) | ((m_0.x & 0x8000u) ? one << 16 : 0u);
            o0.w = static_cast<unsigned>(bf16_bits(ch6)) | (static_cast<unsigned>(bf16_bits(ch7)) << 16);
            o1.x = ((ta >> 16) ? one : 0u) | ((tb >> 16) ? one << 16 : 0u);
            o1.y = ((ta & 1u) ? one : 0u) | ((tb & 1u) ? one << 16 : 0u);
            o1.z = 0u;
            o1.w = 0u;
            const long i = x + static_cast<long>(gr.nx) * y + static_cast<long>(gr.nxy) * zc;
            uint4* dst = reinterpret_cast<uint4*>(feat) + 2 * i;
            dst[0] = o0;
            dst[1] = o1;
        }
        sf_m = sf_0, sh_m = sh_0, sf_0 = sf, sh_0 = sh;
        t_0 = t_in, m_0 = c, v_0 = pv[0];
        t_dn = t_hold, t_hold = t_next;  // vertex z + 1 is written when plane z + 2 is in LDS
        if (z < z_end) store(slot ^ 1);
        __syncthreads();
    }
}

// Mean squared error: loss partial sums and dL/dp (the output layer is
// linear), stored as a 16-channel gradient tensor with channel 0 in use.
// Vertex i weighs 1 + edit_weight when its target is positive.
__global__ void __launch_bounds__(256) k_mse(const float* __restrict__ p, const float* __restrict__ target, int n,
                                             float edit_weight, uint16_t* __restrict__ dz,
                                             float* __restrict__ loss_part) {
    __shared__ float red[4];
    float acc = 0.0f;
    const float scale = 2.0f / static_cast<float>(n);
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float t = target[i];
        const float d = p[i] - t;
        const float w = t > 0.0f ? 1.0f + edit_weight : 1.0f;
        acc += w * d * d;
        const float gz = scale * w * d;
        uint4* row = reinterpret_cast<uint4*>(dz) + 2 * static_cast<long>(i);
        row[0] = make_uint4(bf16_bits(gz), 0u, 0u, 0u);
        row[1] = make_uint4(0u, 0u, 0u, 0u);
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) loss_part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Adam (bias-corrected), FP32 master parameters.
__global__ void __launch_bounds__(256) k_adam(float* __restrict__ w, const float* __restrict__ grad,
                                              float* __restrict__ m1, float* __restrict__ m2, int n, float lr, float b1,
                                              float b2, float eps, float c1, float c2) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float g = grad[i];
        const float a = b1 * m1[i] + (1.0f - b1) * g;
        const float b = b2 * m2[i] + (1.0f - b2) * g * g;
        m1[i] = a;
        m2[i] = b;
        w[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
    }
}

// One decreasing edit (Eqs. 2-6 with the float floor L): halfway to the
// floor, snapped to it when float32 rounding would leave g unchanged.
__device__ __forceinline__ float halve_to(float g, float L) {
    const float h = __fmul_rn(__fadd_rn(g, L), 0.5f);
    return h == g ? L : h;
}

// Warm start: fhat halved k times, k = floor(fl(p - p_min)) + 1 clamped to
// [0, kMaxWarmHalvings] (0 where p is not a number).  The floor is formed
// where a value is halved (a few percent of the vertices): for 256^3 54 us,
// where a pass that stored every floor first and this one took 79.
constexpr int kMaxWarmHalvings = 64;
__global__ void __launch_bounds__(256) k_warm_start(const float* __restrict__ p, const float* __restrict__ f,
                                                    const float* __restrict__ fhat, float xi, float p_min, int n,
                                                    float* __restrict__ g0) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float q = floorf(__fsub_rn(p[i], p_min)) + 1.0f;
        const int k = q > 0.0f ? (q < static_cast<float>(kMaxWarmHalvings) ? static_cast<int>(q) : kMaxWarmHalvings) : 0;
        float g = fhat[i];
        if (k > 0) {
            const float l = floor_bound(f[i], xi);
            for (int j = 0; j < k; ++j) g = halve_to(g, l);
        }
        g0[i] = g;
    }
}

// Training target: the number of halvings that take fhat_i to g_i (-1 when
// g_i is not on that chain within kMaxCount steps).
constexpr int kMaxCount = 256;
__global__ void __launch_bounds__(256) k_halvings(const float* __restrict__ f, const float* __restrict__ fhat,
                                                  const float* __restrict__ g, float xi, int n,
                                                  float* __restrict__ k_out) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float gi = g[i], l = floor_bound(f[i], xi);
        float cur = fhat[i];
        int k = 0;
        while (cur > gi && k < kMaxCount) {
            const float nx = halve_to(cur, l);
            if (!(nx < cur)) break;  // at the floor (or an invalid floor): no further progress
            cur = nx;
            ++k;
        }
        k_out[i] = cur == gi ? static_cast<float>(k) : -1.0f;
    }
}

// ------------------------------------------------------------- launchers ---

constexpr int kConvBlocks = 2048;
// Blocks of the convolutions: as many as run at once (two per compute unit by
// LDS), each walking its tiles, so that a block loads its weights once.
constexpr int kTileBlocks = 512;

static int tiles_of(const Grid& gr, int ty, int tz) {
    return ((gr.nx + 15) / 16) * ((gr.ny + ty - 1) / ty) * ((gr.nz + tz - 1) / tz);
}

template <int MODE>
static void launch_conv_t(const uint16_t* in, const Grid& gr, const WeightView& wv, const uint16_t* mask,
                          uint16_t* out16, hipStream_t s) {
    if (gr.nz == 1) {
        const int nt = tiles_of(gr, 32, 1);
        hipLaunchKernelGGL((k_conv<32, 1, MODE>), dim3(nt < kTileBlocks ? nt : kTileBlocks), dim3(256), 0, s, in, gr, wv,
                           mask, out16);
    } else {
        const int nt = tiles_of(gr, 8, 8);
        hipLaunchKernelGGL((k_conv<8, 8, MODE>), dim3(nt < kTileBlocks ? nt : kTileBlocks), dim3(256), 0, s, in, gr, wv,
                           mask, out16);
    }
}

template <int FX, int FY>
static void launch_features_t(const float* f, const float* fhat, const uint8_t* df, const uint8_t* dh, const Grid& gr,
                              float xi, float xi_ch, uint16_t* feat, hipStream_t s) {
    using T = FeatTile<FX, FY>;
    // a tile per block (at most one per vertex), in rows of 2^20 blocks: a
    // grid's row has fewer than 2^32 threads
    const int nt = ((gr.nx + T::X - 1) / T::X) * ((gr.ny + T::Y - 1) / T::Y) * ((gr.nz + kFeatZ - 1) / kFeatZ);
    const int row = std::min(nt, 1 << 20);
    hipLaunchKernelGGL((k_features<FX, FY>), dim3(row, (nt + row - 1) / row), dim3(256), 0, s, f, fhat, df, dh, gr, nt,
                       xi, xi_ch, feat);
}

// Tiles of 32 x 8 columns, but of another shape in fields of so few columns or
// rows that most of such a tile would lie outside them.  Whole calls with
// 32 x 8 tiles and with these: nx = 1 (1000003 rows) 739 and 230 us; nx = 3
// (300001 rows) 282 and 137; nx = 16 (100 planes of 3000 rows) 308 and 297,
// where nx = 20 takes 292 and 299; ny = 1 (nx = 1000003) 231 and 125; ny = 4
// (nx = 300001) 113 and 95, where ny = 5 takes the same.
static void launch_features(const float* f, const float* fhat, const uint8_t* df, const uint8_t* dh, const Grid& gr,
                            float xi, float xi_ch, uint16_t* feat, hipStream_t s) {
    if (gr.nx == 1) launch_features_t<1, 256>(f, fhat, df, dh, gr, xi, xi_ch, feat, s);
    else if (gr.ny == 1) launch_features_t<256, 1>(f, fhat, df, dh, gr, xi, xi_ch, feat, s);
    else if (gr.nx <= 16) launch_features_t<4, 64>(f, fhat, df, dh, gr, xi, xi_ch, feat, s);
    else if (gr.ny <= 4) launch_features_t<128, 2>(f, fhat, df, dh, gr, xi, xi_ch, feat, s);
    else launch_features_t<32, 8>(f, fhat, df, dh, gr, xi, xi_ch, feat, s);
}

// Tiles of a weight gradient: 16 x 8 x 4 vertices (2D: 16 x 16), so that three
// blocks' tiles with their halos share a compute unit's LDS and one block
// stages while another computes.
static int dw_tiles(const Grid& gr) { return gr.nz == 1 ? tiles_of(gr, 16, 1) : tiles_of(gr, 8, 4); }

// The gradient of one layer's weights (n_out output channels stored) and bias,
// by at most max_blocks blocks (and partial sums).
static void launch_dw(const uint16_t* in, const uint16_t* dz, const Grid& gr, float* part, int max_blocks, int n_out,
                      float* gW, float* gb, hipStream_t s) {
    const int nb = std::min(dw_tiles(gr), std::min(kDwBlocks, max_blocks));
    if (gr.nz == 1) hipLaunchKernelGGL((k_conv_dw<16, 1>), dim3(nb), dim3(256), 0, s, in, dz, gr, part);
    else hipLaunchKernelGGL((k_conv_dw<8, 4>), dim3(nb), dim3(256), 0, s, in, dz, gr, part);
    hipLaunchKernelGGL(k_reduce_dw, dim3((kDwSums + 63) / 64), dim3(1024), 0, s, part, nb, n_out, gW, gb);
}

}  // namespace msz

// ================================================================ C ABI ====

namespace msz {
namespace {

size_t a256(size_t b) { return (b + 255) & ~size_t(255); }
bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Net workspace of one field.
struct NetLayout {
    size_t dirs_f, dirs_h, a1, a2, p, dz_a, dz_b, feat, minmax, g0, total;
    int max_parts;  // partial sums of a weight gradient, from feat on
};

NetLayout net_layout(const Grid& gr) {
    const size_t n = static_cast<size_t>(gr.n);
    NetLayout l{};
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t r = o;
        o += a256(b);
        return r;
    };
    l.dirs_f = take(n + 16);
    l.dirs_h = take(n + 16);
    l.a1 = take(n * 32);
    l.a2 = take(n * 32);
    l.p = take(n * 4);
    l.dz_a = take(n * 32);
    l.dz_b = take(n * 32);
    // The partial sums of a gradient, which is given its features, lie over
    // the features and a part of its own: a partial for each tile of the
    // convolutions, half as many as the weight gradient has tiles.
    l.feat = take(n * 32);
    (void)take(static_cast<size_t>(std::min(kDwBlocks, gr.nz == 1 ? tiles_of(gr, 32, 1) : tiles_of(gr, 8, 8))) *
               kDwSums * 4);
    l.max_parts = static_cast<int>(std::min<size_t>(kDwBlocks, (o - l.feat) / (kDwSums * 4)));
    l.minmax = take(kConvBlocks * 2 * 4);
    l.g0 = take(n * 4);
    l.total = o;
    return l;
}

WeightView layer_view(const float* P, int layer) {
    switch (layer) {
        case 0: return {P + kOffW0, P + kOffB0, 256, 16, 1, 16, 16, 0};
        case 1: return {P + kOffW1, P + kOffB1, 256, 16, 1, 16, 16, 0};
        default: return {P + kOffW2, P + kOffB2, 16, 1, 0, 16, 1, 0};
    }
}

// Weights of the backward-data convolution of layer `layer` (transposed, taps flipped).
WeightView layer_back_view(const float* P, int layer) {
    if (layer == 1) return {P + kOffW1, nullptr, 256, 1, 16, 16, 16, 1};
    return {P + kOffW2, nullptr, 16, 0, 1, 1, 16, 1};  // layer 2: one input channel
}

void net_forward(const float* P, const uint16_t* feat, const Grid& gr, uint16_t* a1, uint16_t* a2, float* p,
                 hipStream_t s) {
    launch_conv_t<kConvHidden>(feat, gr, layer_view(P, 0), nullptr, a1, s);
    launch_conv_t<kConvHidden>(a1, gr, layer_view(P, 1), nullptr, a2, s);
    if (gr.nz == 1) {
        const int nt = tiles_of(gr, 32, 1);
        hipLaunchKernelGGL((k_conv_out<32, 1>), dim3(nt < kTileBlocks ? nt : kTileBlocks), dim3(256), 0, s, a2, gr,
                           P + kOffW2, P + kOffB2, p);
    } else {
        const int nt = tiles_of(gr, 8, 8);
        hipLaunchKernelGGL((k_conv_out<8, 8>), dim3(nt < kTileBlocks ? nt : kTileBlocks), dim3(256), 0, s, a2, gr,
                           P + kOffW2, P + kOffB2, p);
    }
}

__global__ void __launch_bounds__(256) k_minmax(const float* __restrict__ f, int n, float* __restrict__ out) {
    __shared__ float smin[4], smax[4];
    float lo = INFINITY, hi = -INFINITY;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        lo = fminf(lo, f[i]);
        hi = fmaxf(hi, f[i]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, o));
        hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if ((threadIdx.x & 63) == 0) smin[threadIdx.x >> 6] = lo, smax[threadIdx.x >> 6] = hi;
    __syncthreads();
    if (threadIdx.x == 0) {
        out[2 * blockIdx.x] = fminf(fminf(smin[0], smin[1]), fminf(smin[2], smin[3]));
        out[2 * blockIdx.x + 1] = fmaxf(fmaxf(smax[0], smax[1]), fmaxf(smax[2], smax[3]));
    }
}

int blocks_n(long n) {
    long b = (n + 255) / 256;
    return static_cast<int>(b < 1 ? 1 : (b > kConvBlocks ? kConvBlocks : b));
}

int features_impl(const float* f, const float* fhat, const Grid& gr, float xi, uint16_t* feat, char* ws,
                  const NetLayout& l, hipStream_t s) {
    if (!(xi > 0.0f) || !(xi <= kValueLimit)) return MSZ_EINVAL;
    uint8_t* df = reinterpret_cast<uint8_t*>(ws + l.dirs_f);
    uint8_t* dh = reinterpret_cast<uint8_t*>(ws + l.dirs_h);
    float* mm = reinterpret_cast<float*>(ws + l.minmax);
    const int nb = blocks_n(gr.n);
    hipLaunchKernelGGL(k_minmax, dim3(nb), dim3(256), 0, s, f, gr.n, mm);
    std::vector<float> host(2 * nb);
    if (hipMemcpyAsync(host.data(), mm, 2 * nb * sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return MSZ_EDEVICE;
    float lo = host[0], hi = host[1];
    for (int b = 1; b < nb; ++b) lo = fminf(lo, host[2 * b]), hi = fmaxf(hi, host[2 * b + 1]);
    const double range = static_cast<double>(hi) - static_cast<double>(lo);
    if (!(range > 0.0) || !std::isfinite(range)) return MSZ_EINVAL;
    const float xi_ch = static_cast<float>(std::log10(static_cast<double>(xi) / range) / 4.0 + 1.0);
    launch_dirs(f, gr, df, nullptr, s);
    launch_dirs(fhat, gr, dh, nullptr, s);
    launch_features(f, fhat, df, dh, gr, xi, xi_ch, feat, s);
    return hipGetLastError() == hipSuccess ? MSZ_OK : MSZ_EDEVICE;
}

}  // namespace
}  // namespace msz

using namespace msz;

extern "C" {

size_t msz_net_workspace_bytes(msz_dims d) {
    Grid gr;
    if (!make_grid(d, gr)) return 0;
    return net_layout(gr).total;
}

size_t msz_learned_workspace_bytes(msz_dims d) {
    const size_t a = msz_net_workspace_bytes(d), b = msz_workspace_bytes(d);
    return a && b ? a256(a) + b : 0;
}

int msz_net_features(const float* f, const float* fhat, msz_dims d, float xi, uint16_t* feat, void* workspace,
                     size_t workspace_bytes, void* stream) {
    Grid gr;
    if (!make_grid(d, gr) || !f || !fhat || !feat || !al16(feat)) return MSZ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const NetLayout l = net_layout(gr);
    Scratch ws;
    if (int rc = ws.get(workspace, workspace_bytes, l.total, s)) return rc;
    const int rc = features_impl(f, fhat, gr, xi, feat, static_cast<char*>(ws.p), l, s);
    if (rc) return rc;
    return hipStreamSynchronize(s) == hipSuccess ? MSZ_OK : MSZ_EDEVICE;
}

int msz_net_halvings(const float* f, const float* fhat, const float* g, msz_dims d, float xi, float* k_out,
                     void* workspace, size_t workspace_bytes, void* stream) {
    Grid gr;
    if (!make_grid(d, gr) || !f || !fhat || !g || !k_out) return MSZ_EINVAL;
    if (!(xi > 0.0f) || !(xi <= kValueLimit)) return MSZ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // the declared scratch is not needed (the floors are formed in place)
    if (workspace && workspace_bytes < a256(static_cast<size_t>(gr.n) * sizeof(float))) return MSZ_EINVAL;
    hipLaunchKernelGGL(k_halvings, dim3(blocks_n(gr.n)), dim3(256), 0, s, f, fhat, g, xi, gr.n, k_out);
    if (hipGetLastError() != hipSuccess) return MSZ_EDEVICE;
    return hipStreamSynchronize(s) == hipSuccess ? MSZ_OK : MSZ_EDEVICE;
}

int msz_net_forward(const float* params, const uint16_t* feat, msz_dims d, float* p_out, uint16_t* act1_out,
                    uint16_t* act2_out, void* workspace, size_t workspace_bytes, void* stream) {
    Grid gr;
    if (!make_grid(d, gr) || !params || !feat || !p_out || !al16(feat) || !al16(act1_out) || !al16(act2_out))
        return MSZ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const NetLayout l = net_layout(gr);
    Scratch ws;
    if (int rc = ws.get(workspace, workspace_bytes, l.total, s)) return rc;
    char* w = static_cast<char*>(ws.p);
    uint16_t* a1 = act1_out ? act1_out : reinterpret_cast<uint16_t*>(w + l.a1);
    uint16_t* a2 = act2_out ? act2_out : reinterpret_cast<uint16_t*>(w + l.a2);
    net_forward(params, feat, gr, a1, a2, p_out, s);
    if (hipGetLastError() != hipSuccess) return MSZ_EDEVICE;
    return hipStreamSynchronize(s) == hipSuccess ? MSZ_OK : MSZ_EDEVICE;
}

int msz_net_gradients(const float* params, const uint16_t* feat, const float* target, float edit_weight, msz_dims d,
                      float* grad_out, float* loss_out, void* workspace, size_t workspace_bytes, void* stream) {
    Grid gr;
    if (!make_grid(d, gr) || !params || !feat || !target || !grad_out || !loss_out || !al16(feat)) return MSZ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const NetLayout l = net_layout(gr);
    Scratch ws;
    if (int rc = ws.get(workspace, workspace_bytes, l.total, s)) return rc;
    char* w = static_cast<char*>(ws.p);
    uint16_t* a1 = reinterpret_cast<uint16_t*>(w + l.a1);
    uint16_t* a2 = reinterpret_cast<uint16_t*>(w + l.a2);
    float* p = reinterpret_cast<float*>(w + l.p);
    uint16_t* dza = reinterpret_cast<uint16_t*>(w + l.dz_a);
    uint16_t* dzb = reinterpret_cast<uint16_t*>(w + l.dz_b);
    float* part = reinterpret_cast<float*>(w + l.feat);
    float* lp = reinterpret_cast<float*>(w + l.minmax);
    net_forward(params, feat, gr, a1, a2, p, s);
    const int nb = blocks_n(gr.n);
    hipLaunchKernelGGL(k_mse, dim3(nb), dim3(256), 0, s, p, target, gr.n, edit_weight, dza, lp);
    // layer 2
    launch_dw(a2, dza, gr, part, l.max_parts, 1, grad_out + kOffW2, grad_out + kOffB2, s);
    launch_conv_t<kConvBackData>(dza, gr, layer_back_view(params, 2), a2, dzb, s);
    // layer 1
    launch_dw(a1, dzb, gr, part, l.max_parts, 16, grad_out + kOffW1, grad_out + kOffB1, s);
    launch_conv_t<kConvBackData>(dzb, gr, layer_back_view(params, 1), a1, dza, s);
    // layer 0
    launch_dw(feat, dza, gr, part, l.max_parts, 16, grad_out + kOffW0, grad_out + kOffB0, s);
    if (hipGetLastError() != hipSuccess) return MSZ_EDEVICE;
    std::vector<float> host(nb);
    if (hipMemcpyAsync(host.data(), lp, nb * sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return MSZ_EDEVICE;
    double acc = 0.0;
    for (float v : host) acc += v;
    *loss_out = static_cast<float>(acc / gr.n);
    return MSZ_OK;
}

int msz_net_adam(float* params, const float* grad, float* m, float* v, int32_t n, int32_t step, float lr,
                 void* stream) {
    if (!params || !grad || !m || !v || n <= 0 || step < 1) return MSZ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = static_cast<float>(1.0 - std::pow(0.9, step)), c2 = static_cast<float>(1.0 - std::pow(0.999, step));
    hipLaunchKernelGGL(k_adam, dim3(blocks_n(n)), dim3(256), 0, s, params, grad, m, v, n, lr, b1, b2, 1e-8f, c1, c2);
    if (hipGetLastError() != hipSuccess) return MSZ_EDEVICE;
    return hipStreamSynchronize(s) == hipSuccess ? MSZ_OK : MSZ_EDEVICE;
}

int msz_fix_learned(const float* f, const float* fhat, msz_dims d, float xi, const float* params, float p_min,
                    float* edits_out, const msz_options* opt, msz_stats* stats, void* stream) {
    if (!stats) return MSZ_EINVAL;
    std::memset(stats, 0, sizeof(*stats));
    Grid gr;
    msz_options o{};
    if (opt) o = *opt;
    if (!make_grid(d, gr) || !f || !fhat || !params || !edits_out || o.warm_start || !al16(f) || !al16(fhat)) {
        stats->status = MSZ_EINVAL;
        return MSZ_EINVAL;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const NetLayout l = net_layout(gr);
    const size_t fix_bytes = msz_workspace_bytes(d);
    Scratch ws;
    if (int rc = ws.get(o.workspace, o.workspace_bytes, a256(l.total) + fix_bytes, s)) {
        stats->status = rc;
        return rc;
    }
    char* w = static_cast<char*>(ws.p);
    const bool timing = (o.flags & MSZ_FLAG_TIMING) != 0;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (timing && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)) return MSZ_EDEVICE;
    if (timing) (void)hipEventRecord(e0, s);
    uint16_t* feat = reinterpret_cast<uint16_t*>(w + l.feat);
    int rc = features_impl(f, fhat, gr, xi, feat, w, l, s);
    float* p = reinterpret_cast<float*>(w + l.p);
    float* g0 = reinterpret_cast<float*>(w + l.g0);
    if (rc == MSZ_OK) {
        net_forward(params, feat, gr, reinterpret_cast<uint16_t*>(w + l.a1), reinterpret_cast<uint16_t*>(w + l.a2), p, s);
        hipLaunchKernelGGL(k_warm_start, dim3(blocks_n(gr.n)), dim3(256), 0, s, p, f, fhat, xi, p_min, gr.n, g0);
        if (hipGetLastError() != hipSuccess) rc = MSZ_EDEVICE;
    }
    if (timing) (void)hipEventRecord(e1, s);
    if (rc == MSZ_OK) {
        msz_options fo = o;
        fo.warm_start = g0;
        fo.workspace = w + a256(l.total);
        fo.workspace_bytes = fix_bytes;
        rc = msz_fix(f, fhat, d, xi, edits_out, &fo, stats, stream);
    } else {
        stats->status = rc;
    }
    if (timing) {
        float ms = 0.f;
        if (hipEventSynchronize(e1) == hipSuccess && hipEventElapsedTime(&ms, e0, e1) == hipSuccess) {
            stats->phase_ms[MSZ_PHASE_NET] = ms;
            stats->phase_launches[MSZ_PHASE_NET] = 1;
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    return rc;
}

}  // extern "C"
