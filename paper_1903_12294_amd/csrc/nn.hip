// Brick-activity predictor: a 3-layer 3D convolutional network over the grid of
// 8^3-voxel bricks of each timestep, trained on the grower's own results and
// used by the learned scheduler (score order of the tiles, which candidate
// tiles are tested before the rounds).
//
// Activations are channels-last [N][D][H][W][16].  A layer is a 3x3x3
// convolution with zero padding on the gfx950 matrix cores
// (v_mfma_f32_16x16x32_bf16): for 16 input channels one instruction takes two
// kernel offsets x 16 channels (14 per output tile of 16 positions x 16
// channels, the last half empty); the first layer reads only its 8 real
// input channels, four offsets x 8 channels per instruction (7 per tile).
// Weights are bf16, accumulation fp32.
//
// Two precisions of the activations:
//   inference (the scheduler's scores): bf16 activations, one bf16 operand;
//   training (gradients): fp32 activations and fp32 layer gradients.  A
//   convolution splits each fp32 operand into three bf16 pieces (all 24
//   significant bits), so its pre-activations, and the ReLU decisions taken
//   on them, are as accurate as fp32 arithmetic; a weight gradient splits
//   both operands into high part and remainder (hi*hi + hi*lo + lo*hi, about
//   16 bits).  The gradients then follow the fp64 reference element by
//   element.
// The input-gradient of a layer is the same convolution with transposed,
// point-reflected weights; the weight gradient is a reduction over positions
// on the same matrix cores, per block, then summed in a fixed order
// (deterministic).  Parameters are fp32 masters updated by Adam.
#include "nn.h"

#include <algorithm>

namespace mf4d {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// fp32 -> bf16, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ v4f mfma(const uint4& a, const uint4& b, v4f acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                   acc, 0, 0, 0);
}

__device__ __forceinline__ uint4 pack8(const uint16_t* h) {
    return make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}

// Eight fp32 values in three bf16 pieces (high part, then the exact fp32
// remainder split once more): all 24 significant bits, so that a convolution
// of these operands with fp32 accumulation is as accurate as fp32 arithmetic.
__device__ __forceinline__ void split8x3(const float* v, uint4& hi, uint4& mid, uint4& lo) {
    uint16_t h[8], m[8], l[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        h[e] = f2bf(v[e]);
        const float r = v[e] - bf2f(h[e]);
        m[e] = f2bf(r);
        l[e] = f2bf(r - bf2f(m[e]));
    }
    hi = pack8(h);
    mid = pack8(m);
    lo = pack8(l);
}

constexpr int TX = 16, TY = 4, TZ = 4;                  // output positions per block
constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2;   // with halo
constexpr int kHalo = HX * HY * HZ;                    // 648
constexpr int kTilePos = TX * TY * TZ;                 // 256

struct ConvDims {
    int N, D, H, W;
    int nbx, nby, nbz;  // blocks per axis
};

__device__ __forceinline__ void block_origin(const ConvDims& c, uint32_t blk, int& n, int& z0,
                                             int& y0, int& x0) {
    x0 = (blk % c.nbx) * TX;
    blk /= c.nbx;
    y0 = (blk % c.nby) * TY;
    blk /= c.nby;
    z0 = (blk % c.nbz) * TZ;
    n = blk / c.nbz;
}

// Kernel offset k = (dz + 1) * 9 + (dy + 1) * 3 + (dx + 1).
__device__ __forceinline__ int halo_shift(int k) {
    const int dz = k / 9 - 1, dy = (k / 3) % 3 - 1, dx = k % 3 - 1;
    return (dz * HY + dy) * HX + dx;
}

// Matrix operand pieces of an activation type: bf16 as it is, fp32 in three.
template <class T>
constexpr int pieces() { return sizeof(T) == 4 ? 3 : 1; }

// The (TZ+2)(TY+2)(TX+2)-position input tile, CIN channels of each position (of
// the 16 stored), zero outside the grid, staged as matrix operands: plane (piece,
// 8-channel half) holds 16 bytes (8 bf16) per position, so the 16 positions an
// instruction reads lie side by side (no bank conflict), and an fp32 value is
// split here, once, not again for each of the 27 offsets.  A block of 256
// threads; each owns the same places of every tile, so their addresses are
// worked out once and a tile's values can be loaded ahead into registers.
// T = uint16_t (bf16) or float.
template <int CIN, class T>
struct Halo {
    static constexpr int kHalf = CIN / 8, kItems = kHalo * kHalf, kPer = (kItems + 255) / 256;
    static constexpr int kVec = sizeof(T) * 8 / 16;  // 16-byte loads per item
    int rel[kPer];      // positions from the tile's first one (inside the grid below 2^31, as all are)
    uint32_t at[kPer];  // hx, hy, hz (8 bits each), 1 << 24: none
    uint4 val[kPer * kVec];

    __device__ __forceinline__ void init(const ConvDims& c) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = threadIdx.x + u * 256;
            const int p = i / kHalf;
            const int hx = p % HX, hy = (p / HX) % HY, hz = p / (HX * HY);
            rel[u] = (int)(((uint32_t)(hz - 1) * c.H + hy - 1) * c.W + hx - 1);
            at[u] = i < kItems ? hx | (hy << 8) | (hz << 16) : 1u << 24;
        }
    }
    __device__ __forceinline__ void load(const ConvDims& c, const T* __restrict__ x, int n, int z0, int y0, int x0) {
        // (256 is a multiple of kHalf: a thread's items are all of one half)
        const T* base = x + ((((size_t)n * c.D + z0) * c.H + y0) * c.W + x0) * 16 + threadIdx.x % kHalf * 8;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const uint32_t hx = at[u] & 255u, hy = (at[u] >> 8) & 255u, hz = at[u] >> 16;
            const bool in = (uint32_t)(x0 - 1) + hx < (uint32_t)c.W && (uint32_t)(y0 - 1) + hy < (uint32_t)c.H &&
                            hz < 256u && (uint32_t)(z0 - 1) + hz < (uint32_t)c.D;
#pragma unroll
            for (int e = 0; e < kVec; ++e) val[u * kVec + e] = make_uint4(0, 0, 0, 0);
            if (in) {
                const uint4* src = reinterpret_cast<const uint4*>(base + (int64_t)rel[u] * 16);
#pragma unroll
                for (int e = 0; e < kVec; ++e) val[u * kVec + e] = src[e];
            }
        }
    }
    __device__ __forceinline__ void stage(uint4* s_x) const {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = threadIdx.x + u * 256;
            if (i >= kItems) continue;
            const int p = i / kHalf, v = i % kHalf;
            if constexpr (sizeof(T) == 4) {
                const uint4 a = val[2 * u], b = val[2 * u + 1];
                const float f[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z),
                                    __uint_as_float(a.w), __uint_as_float(b.x), __uint_as_float(b.y),
                                    __uint_as_float(b.z), __uint_as_float(b.w)};
                uint4 hi, mid, lo;
                split8x3(f, hi, mid, lo);
                s_x[v * kHalo + p] = hi;
                s_x[(kHalf + v) * kHalo + p] = mid;
                s_x[(2 * kHalf + v) * kHalo + p] = lo;
            } else {
                s_x[v * kHalo + p] = val[u];
            }
        }
    }
};

// Instructions per 16 x 16 output tile: two offsets x 16 channels or four
// offsets x 8 channels each.
template <int CIN>
constexpr int ksteps() { return CIN == 16 ? 14 : 7; }

// (kernel offset, first channel) of the operand lane group g takes in step j;
// offset 27 does not exist (that part of the operand is zero).
template <int CIN>
__device__ __forceinline__ void step_part(int j, int g, int& k, int& c0) {
    if (CIN == 16) {
        k = 2 * j + (g >> 1);
        c0 = 8 * (g & 1);
    } else {
        k = 4 * j + g;
        c0 = 0;
    }
}

enum ConvOut : int { OUT_BF16 = 0, OUT_F32 = 1 };

// out = conv(x, w) + bias, optionally ReLU, optionally zero where mask <= 0
// (mask: the layer's forward activation, fp32 [..][16]: the ReLU derivative).
// x: T [..][16], CIN channels read; fp32 inputs as three bf16 operands.  wpk:
// packed weight operands, [ksteps][64 lanes] x 16 bytes.  Output OUT_BF16: bf16
// [..][16]; OUT_F32: fp32 [..][16] (16-byte stores with vec, else one value at
// a time for a caller's unaligned buffer).
//
// The weights are the first operand, the positions the second: a lane then
// holds four consecutive channels of one position, and a wave stores 16 whole
// positions (512 bytes bf16, 1 KB fp32) in one instruction.  A wave takes the four
// rows of one y, four independent chains, whose LDS addresses differ by constants:
// no address arithmetic between its multiplies.  A block goes over several tiles,
// loading the next one's values while it multiplies; the blocks of an XCD (every
// eighth) take neighbouring tiles, whose halos then meet in its L2.  Bound by the
// LDS reads (1 KB a multiply) and, at the largest, the activations' traffic.
// 64 x 32^3, layers 1 and 2: 30 and 49 us; 48 and 66 with a block per tile and the
// addresses worked out per multiply.
template <int CIN, class T, int OUT>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 2 : 3) void k_conv(ConvDims c, const T* __restrict__ x, const uint4* __restrict__ wpk,
                                              const float* __restrict__ bias, int relu,
                                              const float* __restrict__ mask, void* __restrict__ out, int vec) {
    constexpr int NP = pieces<T>(), NK = ksteps<CIN>(), kHalf = CIN / 8;
    __shared__ uint4 s_x[NP * kHalf * kHalo];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    uint4 bw[NK];
    const uint4* op[NK];  // this lane's operand of each step in the row z = 0
#pragma unroll
    for (int j = 0; j < NK; ++j) {
        int k, c0;
        step_part<CIN>(j, grp, k, c0);
        bw[j] = wpk[j * 64 + lane];
        op[j] = s_x + (c0 >> 3) * kHalo + (HY + wave + 1) * HX + row + 1 + halo_shift(k < 27 ? k : 26);
    }
    int k_last, c_last;
    step_part<CIN>(NK - 1, grp, k_last, c_last);
    v4f b = {0.0f, 0.0f, 0.0f, 0.0f};
    if (bias)
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = bias[4 * grp + i];
    const uint32_t nblocks = (uint32_t)c.N * c.nbz * c.nby * c.nbx;
    // XCD i % 8 takes the tiles [i * per, (i + 1) * per)
    const uint32_t per = (nblocks + 7) / 8, first = (blockIdx.x & 7) * per;
    const uint32_t last = first + per < nblocks ? first + per : nblocks, step = gridDim.x >> 3;
    uint32_t blk = first + (blockIdx.x >> 3);
    if (blk >= last) return;  // block-uniform
    Halo<CIN, T> halo;
    halo.init(c);
    int n, z0, y0, x0;
    block_origin(c, blk, n, z0, y0, x0);
    halo.load(c, x, n, z0, y0, x0);
    while (true) {
        __syncthreads();
        halo.stage(s_x);
        __syncthreads();
        const int zb = z0, yb = y0, xb = x0;
        const size_t pos0 = (((size_t)n * c.D + z0) * c.H + y0) * c.W + x0;
        blk += step;
        const bool more = blk < last;  // block-uniform
        if (more) {
            block_origin(c, blk, n, z0, y0, x0);
            halo.load(c, x, n, z0, y0, x0);
        }
        v4f acc[TZ];
#pragma unroll
        for (int i = 0; i < TZ; ++i) acc[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < NK; ++j)
#pragma unroll
            for (int q = 0; q < NP; ++q)
#pragma unroll
                for (int i = 0; i < TZ; ++i) {
                    uint4 a = op[j][q * kHalf * kHalo + i * HY * HX];
                    if (j == NK - 1 && k_last >= 27) a = make_uint4(0, 0, 0, 0);
                    acc[i] = mfma(bw[j], a, acc[i]);
                }
        // acc[i][e] = D[output channel 4*grp + e][position (zb + i, yb + wave, xb + row)]
        if (yb + wave < c.H && xb + row < c.W) {
#pragma unroll
            for (int i = 0; i < TZ; ++i) {
                if (zb + i >= c.D) break;
                const size_t pos = pos0 + ((uint32_t)(i * c.H + wave) * (uint32_t)c.W + row);
                v4f r = acc[i] + b;
                if (relu)
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[e] = fmaxf(r[e], 0.0f);
                if (mask) {
                    const v4f m = *reinterpret_cast<const v4f*>(mask + pos * 16 + 4 * grp);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (!(m[e] > 0.0f)) r[e] = 0.0f;
                }
                if (OUT == OUT_BF16) {
                    const bf16x4 h = __builtin_convertvector(r, bf16x4);  // to nearest even
                    *reinterpret_cast<bf16x4*>(static_cast<uint16_t*>(out) + pos * 16 + 4 * grp) = h;
                } else {
                    float* o = static_cast<float*>(out) + pos * 16 + 4 * grp;
                    if (vec) {
                        *reinterpret_cast<v4f*>(o) = r;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = r[e];
                    }
                }
            }
        }
        if (!more) break;
    }
}

// The last layer, one output channel: out[position] (fp32 [N][D][H][W]) = conv(x, w)
// + bias over 16 channels.  As 16 output channels of which one is real it would
// take 14 multiplies, each reading 1 KB of LDS, for 16 positions.  Here the rows of
// the first operand are the nine (dz, dy) instead (row 4 (dz + 1) + dy + 1), its
// columns dx and the channels: two multiplies give a row of 16 positions' part of
// all nine, 72 a tile instead of 224.  A wave goes over the rows y of one z and
// adds the parts of dy in registers; those of dz, one in each group of 16 lanes,
// meet in LDS.  wpk: the operand of k_conv (offset k, channels 8h ..: step k / 2, lane
// 32 (k & 1) + 16 h).  Tiles, blocks and loads ahead as in k_conv.
// 64 x 32^3: 27 us, 42 as one of 16 channels.
template <class T>
__global__ __launch_bounds__(256) void k_logit(ConvDims c, const T* __restrict__ x, const uint4* __restrict__ wpk,
                                               const float* __restrict__ bias, float* __restrict__ out) {
    constexpr int NP = pieces<T>();
    __shared__ uint4 s_x[NP * 2 * kHalo];
    __shared__ float s_o[HZ][3][TY][TX];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4, half = grp & 1;
    // step 0: dx = -1 (groups 0, 1) and 0 (groups 2, 3); step 1: dx = 1 (groups 0, 1)
    const int dxi[2] = {grp >> 1, 2};
    uint4 bw[2];
    const uint4* op[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const bool real = row >> 2 < 3 && (row & 3) < 3 && (j == 0 || grp < 2);
        const int k = (row >> 2) * 9 + (row & 3) * 3 + dxi[j];
        bw[j] = real ? wpk[(k >> 1) * 64 + (k & 1) * 32 + half * 16] : make_uint4(0, 0, 0, 0);
        op[j] = s_x + half * kHalo + row + dxi[j];
    }
    const float b = bias[0];
    const uint32_t nblocks = (uint32_t)c.N * c.nbz * c.nby * c.nbx;
    const uint32_t per = (nblocks + 7) / 8, first = (blockIdx.x & 7) * per;
    const uint32_t last = first + per < nblocks ? first + per : nblocks, step = gridDim.x >> 3;
    uint32_t blk = first + (blockIdx.x >> 3);
    if (blk >= last) return;  // block-uniform
    Halo<16, T> halo;
    halo.init(c);
    int n, z0, y0, x0;
    block_origin(c, blk, n, z0, y0, x0);
    halo.load(c, x, n, z0, y0, x0);
    while (true) {
        __syncthreads();
        halo.stage(s_x);
        __syncthreads();
        const int zb = z0, yb = y0, xb = x0;
        const size_t pos0 = (((size_t)n * c.D + z0) * c.H + y0) * c.W + x0;
        blk += step;
        const bool more = blk < last;  // block-uniform
        if (more) {
            block_origin(c, blk, n, z0, y0, x0);
            halo.load(c, x, n, z0, y0, x0);
        }
        for (int hz = wave; hz < HZ; hz += 4) {  // wave-uniform
            v4f acc[HY];
#pragma unroll
            for (int hy = 0; hy < HY; ++hy) acc[hy] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < NP; ++q)
#pragma unroll
                    for (int hy = 0; hy < HY; ++hy) {
                        uint4 a = op[j][q * 2 * kHalo + (hz * HY + hy) * HX];
                        if (j == 1 && grp >= 2) a = make_uint4(0, 0, 0, 0);
                        acc[hy] = mfma(bw[j], a, acc[hy]);
                    }
            // acc[hy][i]: dy = i - 1, dz = grp - 1 of the row (hz, hy): for output y = hy - i, z = hz - grp
            if (grp < 3)
#pragma unroll
                for (int y = 0; y < TY; ++y) s_o[hz][grp][y][row] = (acc[y][0] + acc[y + 1][1]) + acc[y + 2][2];
        }
        __syncthreads();
        const int z = zb + wave, y = yb + grp, xx = xb + row;  // a position a thread
        if (z < c.D && y < c.H && xx < c.W)
            out[pos0 + ((uint32_t)(wave * c.H + grp) * (uint32_t)c.W + row)] =
                ((s_o[wave][0][grp][row] + s_o[wave + 1][1][grp][row]) + s_o[wave + 2][2][grp][row]) + b;
        if (!more) break;
    }
}

// Weight and bias gradients of one layer, per block:
// part_w[blk][k][out][in] = sum_pos dz[pos][out] * x[pos + off(k)][in],
// part_b[blk][out] = sum_pos dz[pos][out], over the tiles blk, blk + gridDim.x,
// ... of 16 x 4 x 4 positions (at most kMaxParts blocks, so that many partials
// whatever the grid).  dz: fp32 [..][16] (COUT channels real); x: T [..][16], CIN
// channels read.  Positions are the reduction axis: one instruction takes 32
// positions (two rows of the tile); each fp32 operand is split into bf16 high
// part and remainder.
//
// Both operands want eight consecutive positions of one channel, so a tile is
// staged channel-major (transposed and split while staging, once per value), and
// wave w owns the kernel offsets (dz, dy) = w of the nine: it reads the ten
// values x - 1 .. x + 8 of a row once and forms the operands of dx = -1, 0, 1
// from them by funnel shifts.  Channel rows are padded so that 8 lanes reading
// 16 bytes of 8 channels hit different banks.  Bound by the staging's latency and
// LDS writes: 19 us for 16 fp32 channels at 32 x 16^3 positions; gathering the
// values one by one and splitting them again for every offset took 51 us.
constexpr int kWX = 24;                                  // LDS row: 18 positions, padded to 16-byte steps
constexpr int kWPlane = HY * HZ * kWX + 8;               // elements per channel
constexpr int kDPlane = kTilePos + 8;
constexpr int kWgradBlock = 9 * 64;
constexpr uint32_t kMaxParts = 1024;  // two resident blocks per CU, twice

// Elements 0..9 (w: 0..7, t: 8, 9) of eight bf16 pairs; the eight starting at S.
template <int S>
__device__ __forceinline__ uint4 window(const uint4& w, uint32_t t) {
    if (S == 0) return w;
    if (S == 2) return make_uint4(w.y, w.z, w.w, t);
    return make_uint4(__builtin_amdgcn_alignbit(w.y, w.x, 16), __builtin_amdgcn_alignbit(w.z, w.y, 16),
                      __builtin_amdgcn_alignbit(w.w, w.z, 16), __builtin_amdgcn_alignbit(t, w.w, 16));
}

template <int CIN, class T>
__global__ __launch_bounds__(kWgradBlock) void k_wgrad(ConvDims c, const T* __restrict__ x,
                                                       const float* __restrict__ dz, float* __restrict__ part_w,
                                                       float* __restrict__ part_b) {
    constexpr bool kF32 = sizeof(T) == 4;
    constexpr int NX = kF32 ? 2 : 1;                     // operand pieces of x
    __shared__ __align__(16) uint16_t s_x[NX * CIN * kWPlane];
    __shared__ __align__(16) uint16_t s_d[2 * 16 * kDPlane];
    __shared__ float s_b[9][16];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    v4f acc[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) acc[j] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
    float bsum[4] = {0.0f, 0.0f, 0.0f, 0.0f};            // channels 4 * (thread & 3) ..
    const uint32_t nblocks = (uint32_t)c.N * c.nbz * c.nby * c.nbx;
    for (uint32_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        int n, z0, y0, x0;
        block_origin(c, blk, n, z0, y0, x0);
        __syncthreads();  // the previous tile's reads are done
        // x: a thread takes 4 channels of two neighbouring positions (one word
        // per channel and piece)
        constexpr int kQuads = CIN / 4, kPairs = HX / 2;
        for (int i = threadIdx.x; i < HZ * HY * kPairs * kQuads; i += kWgradBlock) {
            const int v = i % kQuads, r = i / kQuads;
            const int px = (r % kPairs) * 2, rz = r / kPairs;  // rz = hz * HY + hy
            const int zz = z0 + rz / HY - 1, yy = y0 + rz % HY - 1;
            const bool inr = zz >= 0 && zz < c.D && yy >= 0 && yy < c.H;
            uint16_t h[2][4] = {}, l[2][4] = {};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int xx = x0 + px + e - 1;
                if (!inr || xx < 0 || xx >= c.W) continue;
                const T* src = x + ((((size_t)n * c.D + zz) * c.H + yy) * c.W + xx) * 16 + v * 4;
                if constexpr (kF32) {
                    const float4 u = *reinterpret_cast<const float4*>(src);
                    const float f[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        h[e][q] = f2bf(f[q]);
                        l[e][q] = f2bf(f[q] - bf2f(h[e][q]));
                    }
                } else {
                    const uint2 u = *reinterpret_cast<const uint2*>(src);
                    h[e][0] = (uint16_t)u.x;
                    h[e][1] = (uint16_t)(u.x >> 16);
                    h[e][2] = (uint16_t)u.y;
                    h[e][3] = (uint16_t)(u.y >> 16);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = (v * 4 + q) * kWPlane + rz * kWX + px;
                *reinterpret_cast<uint32_t*>(&s_x[at]) = h[0][q] | ((uint32_t)h[1][q] << 16);
                if (kF32) *reinterpret_cast<uint32_t*>(&s_x[CIN * kWPlane + at]) = l[0][q] | ((uint32_t)l[1][q] << 16);
            }
        }
        // dz: likewise, pairs of positions along x
        for (int i = threadIdx.x; i < kTilePos / 2 * 4; i += kWgradBlock) {
            const int v = i & 3, p = (i >> 2) * 2;
            const int px = p % TX, py = (p / TX) % TY, pz = p / (TX * TY);
            const int zz = z0 + pz, yy = y0 + py;
            uint16_t h[2][4] = {}, l[2][4] = {};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int xx = x0 + px + e;
                if (zz >= c.D || yy >= c.H || xx >= c.W) continue;
                const float4 u =
                    *reinterpret_cast<const float4*>(dz + ((((size_t)n * c.D + zz) * c.H + yy) * c.W + xx) * 16 + v * 4);
                const float f[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    h[e][q] = f2bf(f[q]);
                    l[e][q] = f2bf(f[q] - bf2f(h[e][q]));
                    bsum[q] += f[q];
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = (v * 4 + q) * kDPlane + p;
                *reinterpret_cast<uint32_t*>(&s_d[at]) = h[0][q] | ((uint32_t)h[1][q] << 16);
                *reinterpret_cast<uint32_t*>(&s_d[16 * kDPlane + at]) = l[0][q] | ((uint32_t)l[1][q] << 16);
            }
        }
        __syncthreads();
        const int ch = row < CIN ? row : 0;              // lanes past the channels read zeros (below)
        const int oz = wave / 3, oy = wave % 3;          // dz + 1, dy + 1
#pragma unroll
        for (int k = 0; k < kTilePos / 32; ++k) {
            // positions 32 k + 8 grp + e: row 2 k + (grp >> 1) of the tile, x = 8 (grp & 1) + e
            const int r = 2 * k + (grp >> 1), px = 8 * (grp & 1);
            const int dat = row * kDPlane + r * TX + px;
            const uint4 ahi = *reinterpret_cast<const uint4*>(&s_d[dat]);
            const uint4 alo = *reinterpret_cast<const uint4*>(&s_d[16 * kDPlane + dat]);
            const int xat = ch * kWPlane + ((r / TY + oz) * HY + r % TY + oy) * kWX + px;
            uint4 w[NX];
            uint32_t t[NX];
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                w[q] = *reinterpret_cast<const uint4*>(&s_x[q * CIN * kWPlane + xat]);
                t[q] = *reinterpret_cast<const uint32_t*>(&s_x[q * CIN * kWPlane + xat + 8]);
                if (row >= CIN) {
                    w[q] = make_uint4(0, 0, 0, 0);
                    t[q] = 0;
                }
            }
            auto step = [&](v4f& a, const uint4& bhi, const uint4& blo) {
                a = mfma(ahi, bhi, a);
                a = mfma(alo, bhi, a);
                if (kF32) a = mfma(ahi, blo, a);
            };
            step(acc[0], window<0>(w[0], t[0]), window<0>(w[NX - 1], t[NX - 1]));
            step(acc[1], window<1>(w[0], t[0]), window<1>(w[NX - 1], t[NX - 1]));
            step(acc[2], window<2>(w[0], t[0]), window<2>(w[NX - 1], t[NX - 1]));
        }
    }
    // acc[j][i] = D[out = 4*grp + i][in = row] of offset 3 * wave + j
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            part_w[(((size_t)blockIdx.x * 27 + 3 * wave + j) * 16 + 4 * grp + i) * 16 + row] = acc[j][i];
    // channel sums: lanes with the same thread & 3 hold the same channels
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        for (int o = 4; o < 64; o <<= 1) bsum[q] += __shfl_xor(bsum[q], o);
        if (lane < 4) s_b[wave][lane * 4 + q] = bsum[q];
    }
    __syncthreads();
    if (threadIdx.x < 16) {
        float s = 0.0f;
        for (int w = 0; w < 9; ++w) s += s_b[w][threadIdx.x];
        part_b[(size_t)blockIdx.x * 16 + threadIdx.x] = s;
    }
}

// Block partials of one layer -> its gradients in the reference layout, each sum
// in a fixed order (deterministic): weight i = (k, out, in), then the biases,
// then (loss non-null) the mean loss from part_loss.  A block takes 32
// neighbouring sums (128 bytes of each partial) and splits their partials over 8
// groups of lanes, so a sum is 8 chains of nblk / 8 loads, 8 of them in flight,
// instead of one chain of nblk: bound by the latency of those loads.  A training
// pass with 512 partials per layer (32 x 16^3 positions) went from 1,031 us (one
// thread per sum: 592 us of it, biases, loss and reordering in launches of their
// own) to 440 us.
constexpr int kRedCols = 32, kRedRows = 8;
__global__ __launch_bounds__(kRedCols * kRedRows) void k_reduce_grads(
    const float* __restrict__ part_w, const float* __restrict__ part_b, uint32_t nblk, NetShapes s, int layer,
    float* __restrict__ grads, const float* __restrict__ part_loss, float* __restrict__ loss) {
    __shared__ float s_sum[kRedRows][kRedCols];
    const int cin = s.cin[layer], cout = s.cout[layer];
    const int nw = cout * cin * 27;
    const int col = threadIdx.x % kRedCols, grp = threadIdx.x / kRedCols;
    const int i = blockIdx.x * kRedCols + col;
    const float* src = nullptr;
    float* dst = nullptr;
    size_t stride = 0;
    uint32_t n = nblk;
    if (i < nw) {
        const int ci = i % cin, o = (i / cin) % cout, k = i / (cin * cout);
        src = part_w + (k * 16 + o) * 16 + ci;
        stride = 27 * 256;
        dst = grads + s.woff[layer] + (o * cin + ci) * 27 + k;
    } else if (i < nw + cout) {
        src = part_b + (i - nw);
        stride = 16;
        dst = grads + s.boff[layer] + (i - nw);
    } else if (i == nw + cout && loss) {
        src = part_loss;
        stride = 1;
        n = kLossBlocks;
        dst = loss;
    }
    float acc = 0.0f;
    if (src) {
#pragma unroll 8
        for (uint32_t b = grp; b < n; b += kRedRows) acc += src[b * stride];
    }
    s_sum[grp][col] = acc;
    __syncthreads();
    if (grp == 0 && dst) {
        float v = 0.0f;
        for (int g = 0; g < kRedRows; ++g) v += s_sum[g][col];
        *dst = v;
    }
}

// Binary cross entropy with logits, positive weight pw, mean over n
// positions: dz (fp32 [..][16], channel 0; the rest zero) and per-block
// shares of the mean loss.
__global__ __launch_bounds__(256) void k_bce(const float* __restrict__ logits,
                                             const uint8_t* __restrict__ y, uint64_t n, float pw,
                                             float* __restrict__ dz, float* __restrict__ part_loss) {
    __shared__ float s_sum[4];
    float acc = 0.0f;
    const float inv = 1.0f / (float)n;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const float z = logits[i];
        const float t = y[i] ? 1.0f : 0.0f;
        const float sp_neg = fmaxf(-z, 0.0f) + log1pf(expf(-fabsf(z)));  // softplus(-z)
        const float sp_pos = fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));   // softplus(z)
        acc += pw * t * sp_neg + (1.0f - t) * sp_pos;
        const float s = 1.0f / (1.0f + expf(-z));
        const float g = (s * (pw * t + 1.0f - t) - pw * t) * inv;
        float4* o = reinterpret_cast<float4*>(dz + i * 16);
        o[0] = make_float4(g, 0.f, 0.f, 0.f);
        o[1] = o[2] = o[3] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane_id() == 0) s_sum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part_loss[blockIdx.x] = (s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3]) * inv;
}

// fp32 parameters (reference layout) -> packed bf16 weight operands and biases.
// Forward of layer l (input channels cin_l): W[kappa][out], kappa = (offset,
// input channel) in the order step_part gives.  Input gradient of layer l: the
// convolution of the layer's output gradient (cout_l channels, read as 16, or
// as 8 when cout_l = 1) with W[out][in][26 - k] transposed.
// Slot s: 0..2 forward of layers 0..2, 3..5 input gradient of layers 0..2.
__global__ void k_pack_weights(const float* __restrict__ params, NetShapes sh, uint4* __restrict__ wpk,
                               float* __restrict__ bias) {
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    for (int i = tid; i < 6 * kPackSlot; i += gridDim.x * blockDim.x) {
        const int slot = i / kPackSlot, r = i % kPackSlot;
        const int j = r / 64, lane = r % 64, g = lane >> 4, col = lane & 15;
        const int layer = slot % 3;
        const bool bwd = slot >= 3;
        const int cin = sh.cin[layer], cout = sh.cout[layer];
        const float* W = params + sh.woff[layer];
        // channels the operand reads on its input side
        const int cread = bwd ? (cout == 1 ? 8 : 16) : (cin == 8 ? 8 : 16);
        const int nk = cread == 16 ? 14 : 7;
        uint16_t h[8];
        for (int e = 0; e < 8; ++e) {
            float v = 0.0f;
            if (j < nk) {
                const int k = cread == 16 ? 2 * j + (g >> 1) : 4 * j + g;
                const int ci = (cread == 16 ? 8 * (g & 1) : 0) + e;
                if (k < 27) {
                    if (!bwd && col < cout && ci < cin) v = W[(col * cin + ci) * 27 + k];
                    if (bwd && col < cin && ci < cout) v = W[(ci * cin + col) * 27 + (26 - k)];
                }
            }
            h[e] = f2bf(v);
        }
        wpk[i] = pack8(h);
    }
    for (int i = tid; i < 48; i += gridDim.x * blockDim.x) {
        const int layer = i / 16, o = i % 16;
        bias[i] = o < sh.cout[layer] ? params[sh.boff[layer] + o] : 0.0f;
    }
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

// ---- features and labels from the grower's state ----

// Load time: per brick-step (8^3 voxels of one timestep) min, max, mean of
// the non-NaN field values (-1 for all three when there are none).
__global__ __launch_bounds__(256) void k_brick_stats(Geom g, BrickDims bd, const float* __restrict__ f,
                                                     float4* __restrict__ stats) {
    __shared__ float s_mn[4], s_mx[4], s_sum[4], s_cnt[4];
    const uint32_t b = blockIdx.x;
    const int bx = b % bd.W, by = (b / bd.W) % bd.H, bz = (b / (bd.W * bd.H)) % bd.D,
              t = b / (bd.W * bd.H * bd.D);
    float mn = __builtin_inff(), mx = -__builtin_inff(), sum = 0.0f, cnt = 0.0f;
    for (int i = threadIdx.x; i < 512; i += blockDim.x) {
        const int x = bx * 8 + (i & 7), y = by * 8 + ((i >> 3) & 7), z = bz * 8 + (i >> 6);
        if (x < g.X && y < g.Y && z < g.Z) {
            const float v = f[(((size_t)t * g.Z + z) * g.Y + y) * g.X + x];
            if (v == v) {
                mn = fminf(mn, v);
                mx = fmaxf(mx, v);
                sum += v;
                cnt += 1.0f;
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, o));
        mx = fmaxf(mx, __shfl_xor(mx, o));
        sum += __shfl_xor(sum, o);
        cnt += __shfl_xor(cnt, o);
    }
    if (lane_id() == 0) {
        s_mn[threadIdx.x >> 6] = mn;
        s_mx[threadIdx.x >> 6] = mx;
        s_sum[threadIdx.x >> 6] = sum;
        s_cnt[threadIdx.x >> 6] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        mn = fminf(fminf(s_mn[0], s_mn[1]), fminf(s_mn[2], s_mn[3]));
        mx = fmaxf(fmaxf(s_mx[0], s_mx[1]), fmaxf(s_mx[2], s_mx[3]));
        sum = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
        cnt = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        stats[b] = cnt > 0 ? make_float4(mn, mx, sum / cnt, 0.0f) : make_float4(-1.f, -1.f, -1.f, 0.f);
    }
}

// Load time: particle-steps per brick-step (into stats[].w).
__global__ void k_brick_pcount(Geom g, PGeom pg, BrickDims bd, const uint32_t* __restrict__ bins,
                               float4* __restrict__ stats) {
    const uint64_t n = (uint64_t)pg.P * pg.Tpad;
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < n;
         e += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t b = bins[e];
        if (b == kNoVoxel) continue;
        const uint32_t word = b >> 5;
        const uint32_t tile = word >> (6 + g.logBT);
        const uint32_t wi = word & (g.WPT - 1);
        uint32_t r = tile;
        const int tx = r % g.NXt;
        r /= g.NXt;
        const int ty = r % g.NYt;
        r /= g.NYt;
        const int tz = r % g.NZt;
        const int tt = r / g.NZt;
        const int x = tx * 32 + (b & 31), y = ty * 8 + (wi & 7), z = tz * 8 + ((wi >> 3) & 7);
        const int t = (tt << g.logBT) + (wi >> 6);
        const uint32_t bi = (((uint32_t)t * bd.D + (z >> 3)) * bd.H + (y >> 3)) * bd.W + (x >> 3);
        atomicAdd(&stats[bi].w, 1.0f);
    }
}

// Per grow: network input at brick-step (t, z, y, x): field min / max / mean
// minus the field lower bound and log1p(particle count) / 4, at t and at t-1
// (zeros at t = 0); channels 8..15 zero.
__global__ void k_features(BrickDims bd, const float4* __restrict__ stats, float f_lo,
                           uint16_t* __restrict__ x) {
    const uint64_t n = (uint64_t)bd.T * bd.D * bd.H * bd.W;
    const uint64_t per_t = (uint64_t)bd.D * bd.H * bd.W;
    const float c = (f_lo == f_lo && fabsf(f_lo) < 1e30f) ? f_lo : 0.0f;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t t = i / per_t;
        const float4 s0 = stats[i];
        const float4 s1 = t > 0 ? stats[i - per_t] : make_float4(c, c, c, 0.0f);
        uint16_t v[16];
        v[0] = f2bf(s0.x - c);
        v[1] = f2bf(s0.y - c);
        v[2] = f2bf(s0.z - c);
        v[3] = f2bf(log1pf(s0.w) * 0.25f);
        v[4] = f2bf(s1.x - c);
        v[5] = f2bf(s1.y - c);
        v[6] = f2bf(s1.z - c);
        v[7] = f2bf(log1pf(s1.w) * 0.25f);
        for (int k = 8; k < 16; ++k) v[k] = 0;
        uint4* o = reinterpret_cast<uint4*>(x + i * 16);
        o[0] = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
        o[1] = make_uint4(0, 0, 0, 0);
    }
}

// After a grow: brick-step label = it holds a member voxel.
__global__ void k_brick_labels(Geom g, BrickDims bd, const uint32_t* __restrict__ L,
                               const uint8_t* __restrict__ active, uint8_t* __restrict__ y) {
    const uint64_t n = (uint64_t)bd.T * bd.D * bd.H * bd.W;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const int bx = i % bd.W, by = (i / bd.W) % bd.H, bz = (i / ((uint64_t)bd.W * bd.H)) % bd.D;
        const int t = (int)(i / ((uint64_t)bd.W * bd.H * bd.D));
        const int tx = bx >> 2, xs = (bx & 3) * 8;  // 4 bricks of 8 x-bits per tile word
        const int tt = t >> g.logBT, tl = t & (g.BT - 1);
        const uint32_t tile = ((uint32_t)(tt * g.NZt + bz) * g.NYt + by) * g.NXt + tx;
        uint32_t any = 0;
        if (active[tile]) {
            const uint32_t* w = L + (size_t)tile * g.WPT + tl * 64;
            for (int k = 0; k < 64; ++k) any |= (w[k] >> xs) & 0xFFu;
        }
        y[i] = any ? 1 : 0;
    }
}

// Scores -> tiles to test before the rounds: a candidate tile is tested up
// front when any of its brick-steps scores at least `thr` (logit); the other
// candidates are deferred to the first sweep that reaches them.
__global__ void k_tile_predict(Geom g, BrickDims bd, const float* __restrict__ logits, float thr,
                               uint8_t* __restrict__ pred) {
    for (uint32_t tile = blockIdx.x * blockDim.x + threadIdx.x; tile < g.NT;
         tile += gridDim.x * blockDim.x) {
        uint32_t r = tile;
        const int tx = r % g.NXt;
        r /= g.NXt;
        const int ty = r % g.NYt;
        r /= g.NYt;
        const int tz = r % g.NZt;
        const int tt = r / g.NZt;
        bool hot = false;
        for (int tl = 0; tl < g.BT && !hot; ++tl) {
            const int t = (tt << g.logBT) + tl;
            if (t >= g.T) break;
            for (int k = 0; k < 4; ++k) {
                const int bx = tx * 4 + k;
                if (bx >= bd.W) break;
                const uint64_t i = (((uint64_t)t * bd.D + tz) * bd.H + ty) * bd.W + bx;
                if (logits[i] >= thr) {
                    hot = true;
                    break;
                }
            }
        }
        pred[tile] = hot ? 1 : 0;
    }
}

inline unsigned grid_for(uint64_t n, unsigned block, unsigned cap) {
    uint64_t b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

ConvDims conv_dims(int N, int D, int H, int W) {
    ConvDims c{N, D, H, W, (W + TX - 1) / TX, (H + TY - 1) / TY, (D + TZ - 1) / TZ};
    return c;
}

template <int CIN, class T, int OUT>
void conv_launch(int N, int D, int H, int W, const T* x, const uint4* wpk, const float* bias, int relu,
                 const float* mask, void* out, hipStream_t s) {
    const ConvDims c = conv_dims(N, D, H, W);
    const uint32_t nb = (uint32_t)c.N * c.nbz * c.nby * c.nbx;
    const int vec = (reinterpret_cast<uintptr_t>(out) & 15) == 0;  // a caller's dx may not be
    // blocks in eighths, one to an XCD, as many as are resident at once (bf16 three a CU, fp32 two)
    const unsigned blocks = 8 * grid_for(nb, 8, sizeof(T) == 4 ? 64 : 96);
    hipLaunchKernelGGL((k_conv<CIN, T, OUT>), dim3(blocks), dim3(256), 0, s, c, x, wpk, bias, relu, mask, out, vec);
}

template <class T>
void logit_launch(int N, int D, int H, int W, const T* x, const uint4* wpk, const float* bias, float* out,
                  hipStream_t s) {
    const ConvDims c = conv_dims(N, D, H, W);
    const uint32_t nb = (uint32_t)c.N * c.nbz * c.nby * c.nbx;
    // as many as are resident at once (bf16 four a CU, fp32 two)
    const unsigned blocks = 8 * grid_for(nb, 8, sizeof(T) == 4 ? 64 : 128);
    hipLaunchKernelGGL((k_logit<T>), dim3(blocks), dim3(256), 0, s, c, x, wpk, bias, out);
}

// Gradients of layer `layer` (and, with loss, the mean loss from part_loss).
template <int CIN, class T>
void wgrad_launch(int N, int D, int H, int W, const T* x, const float* dz, float* part_w, float* part_b,
                  const NetShapes& sh, int layer, float* grads, const float* part_loss, float* loss, hipStream_t s) {
    const ConvDims c = conv_dims(N, D, H, W);
    const uint32_t nb = nn_blocks(N, D, H, W);
    hipLaunchKernelGGL((k_wgrad<CIN, T>), dim3(nb), dim3(kWgradBlock), 0, s, c, x, dz, part_w, part_b);
    const int sums = sh.cout[layer] * sh.cin[layer] * 27 + sh.cout[layer] + 1;
    hipLaunchKernelGGL(k_reduce_grads, dim3((sums + kRedCols - 1) / kRedCols), dim3(kRedCols * kRedRows), 0, s,
                       part_w, part_b, nb, sh, layer, grads, part_loss, loss);
}

}  // namespace

uint32_t nn_blocks(int N, int D, int H, int W) {
    const ConvDims c = conv_dims(N, D, H, W);
    return std::min((uint32_t)c.N * c.nbz * c.nby * c.nbx, kMaxParts);
}

void launch_infer(int N, int D, int H, int W, const uint16_t* x, const uint4* wpk, const float* bias,
                  uint16_t* a1, uint16_t* a2, float* logits, hipStream_t s) {
    conv_launch<8, uint16_t, OUT_BF16>(N, D, H, W, x, wpk + 0 * kPackSlot, bias, 1, nullptr, a1, s);
    conv_launch<16, uint16_t, OUT_BF16>(N, D, H, W, a1, wpk + 1 * kPackSlot, bias + 16, 1, nullptr, a2, s);
    logit_launch<uint16_t>(N, D, H, W, a2, wpk + 2 * kPackSlot, bias + 32, logits, s);
}

void launch_train_forward(int N, int D, int H, int W, const uint16_t* x, const uint4* wpk, const float* bias,
                          float* a1, float* a2, float* logits, hipStream_t s) {
    conv_launch<8, uint16_t, OUT_F32>(N, D, H, W, x, wpk + 0 * kPackSlot, bias, 1, nullptr, a1, s);
    conv_launch<16, float, OUT_F32>(N, D, H, W, a1, wpk + 1 * kPackSlot, bias + 16, 1, nullptr, a2, s);
    logit_launch<float>(N, D, H, W, a2, wpk + 2 * kPackSlot, bias + 32, logits, s);
}

void launch_train_backward(int N, int D, int H, int W, const uint16_t* x, const uint4* wpk, const float* logits,
                           const uint8_t* y, float pw, const float* a1, const float* a2, float* dz1, float* dz2,
                           float* dz3, float* dx, float* part_w, float* part_b, float* part_loss, float* loss,
                           const NetShapes& sh, float* grads, hipStream_t s) {
    const uint64_t pos = (uint64_t)N * D * H * W;
    hipLaunchKernelGGL(k_bce, dim3(kLossBlocks), dim3(256), 0, s, logits, y, pos, pw, dz3, part_loss);
    // layer 3: weights from a2 and dz3; dz2 = input gradient masked by relu'(z2)
    wgrad_launch<16, float>(N, D, H, W, a2, dz3, part_w, part_b, sh, 2, grads, part_loss, loss, s);
    conv_launch<8, float, OUT_F32>(N, D, H, W, dz3, wpk + 5 * kPackSlot, nullptr, 0, a2, dz2, s);
    // layer 2
    wgrad_launch<16, float>(N, D, H, W, a1, dz2, part_w, part_b, sh, 1, grads, nullptr, nullptr, s);
    conv_launch<16, float, OUT_F32>(N, D, H, W, dz2, wpk + 4 * kPackSlot, nullptr, 0, a1, dz1, s);
    // layer 1: weights from the bf16 inputs; the input gradient on request
    wgrad_launch<8, uint16_t>(N, D, H, W, x, dz1, part_w, part_b, sh, 0, grads, nullptr, nullptr, s);
    if (dx) conv_launch<16, float, OUT_F32>(N, D, H, W, dz1, wpk + 3 * kPackSlot, nullptr, 0, nullptr, dx, s);
}

void launch_pack_weights(const float* params, const NetShapes& sh, uint4* wpk, float* bias, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_weights, dim3(21), dim3(256), 0, s, params, sh, wpk, bias);
}

void launch_adam(float* p, const float* g, float* m, float* v, int n, float lr, float b1, float b2,
                 float eps, int step, hipStream_t s) {
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n, 256, 64)), dim3(256), 0, s, p, g, m, v, n, lr, b1,
                       b2, eps, c1, c2);
}

void launch_brick_stats(const Geom& g, const PGeom& pg, const BrickDims& bd, const float* field,
                        const uint32_t* bins, float4* stats, hipStream_t s) {
    const uint32_t nb = (uint32_t)((uint64_t)bd.T * bd.D * bd.H * bd.W);
    hipLaunchKernelGGL(k_brick_stats, dim3(nb), dim3(256), 0, s, g, bd, field, stats);
    if (pg.P > 0 && bins)
        hipLaunchKernelGGL(k_brick_pcount, dim3(grid_for((uint64_t)pg.P * pg.Tpad, 256, 8192)),
                           dim3(256), 0, s, g, pg, bd, bins, stats);
}

void launch_features(const BrickDims& bd, const float4* stats, float f_lo, uint16_t* x,
                     hipStream_t s) {
    const uint64_t n = (uint64_t)bd.T * bd.D * bd.H * bd.W;
    hipLaunchKernelGGL(k_features, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, bd, stats, f_lo, x);
}

void launch_brick_labels(const Geom& g, const BrickDims& bd, const uint32_t* L,
                         const uint8_t* active, uint8_t* y, hipStream_t s) {
    const uint64_t n = (uint64_t)bd.T * bd.D * bd.H * bd.W;
    hipLaunchKernelGGL(k_brick_labels, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s, g, bd, L,
                       active, y);
}

void launch_tile_predict(const Geom& g, const BrickDims& bd, const float* logits, float thr,
                         uint8_t* pred, hipStream_t s) {
    hipLaunchKernelGGL(k_tile_predict, dim3(grid_for(g.NT, 256, 4096)), dim3(256), 0, s, g, bd,
                       logits, thr, pred);
}

}  // namespace mf4d
