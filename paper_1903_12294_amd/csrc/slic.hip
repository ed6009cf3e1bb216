// 4D SLIC clustering of point and field samples (Section 3.2) on gfx950.
//
// One iteration is two fused passes (field samples, then point samples) and
// one small update.  A pass assigns each sample to the centre with the
// smallest distance among those whose window holds it (Section 3.2.2-3.2.3)
// and adds the sample's quantised coordinates and value to its centre's
// sums: first block-local in LDS, then with one 64-bit atomic per touched
// centre and sum.  Integer sums make the centres independent of the
// order of the additions, so they are bit-identical run to run.  The update
// turns the sums into means, compares them with the previous centres
// (convergence, Section 3.2.2) and clears the sums.
//
// A block takes a compact box of samples (field: up to 32 x 8 x 8 x 2
// voxel-steps; points: 1,024 consecutive ones in visiting order, sorted by
// sub-box), lists the centres whose windows meet the box, and each wave keeps
// of these, per 256 samples, the ones that can win for any of them (bounds of
// the distance over the wave's box).  A sample so rates about ten centres
// instead of testing the hundreds of its neighbourhood.  Boxes whose list would
// not fit are noted, and a third kernel searches them sample by sample.
//
// Arithmetic that decides a label is fp32 in a fixed order, with the products
// fused into the sums and the hardware's square root (1 ulp):
//   S^2 = (cf*dt)^2 + (dz^2 + (dx^2 + dy^2)),  D = w_v*|v - v_c| + w_d*S,
// dist2 and distance below.  (The oracle rounds every operation on its own: two
// centres whose distances from a sample agree to 2^-20 may rank otherwise there.
// This is the arithmetic that the same distance written with single roundings
// compiles to: the compiler fuses those too.)
#include "slic.h"

#include <math.h>

#include <algorithm>

namespace mf4d {
namespace {

constexpr double kQInv = 1.0 / 1048576.0;
constexpr float kMaxAbs = 2048.0f;     // |coordinate|, |value| below this keep the sums in int64
constexpr int kTab = 64;               // LDS table slots (centres one block touches)
constexpr int kBlock = 256;
constexpr int kPer = 4;                // samples per thread per pass
constexpr int kCand = 256;             // centres a box's list holds (4 per lane of a wave)
constexpr int kAxis = 64;              // slabs per axis a box may meet
constexpr int kRaw = 16384;            // slab combinations tested for a box's list

__device__ __forceinline__ int seed_cell(float pos, float C, int kd) {
    const float q = floorf(__fdiv_rn(pos, C));
    return (int)fminf(fmaxf(q, 0.0f), (float)(kd - 1));
}

// rint(v * 2^20) for |v| < 2048: the product by a power of two is exact in fp32
// and below 2^31.
__device__ __forceinline__ int quantise(float v) { return __float2int_rn(__fmul_rn(v, 1048576.0f)); }

// dbl(s) = float64(s >> 32) * 2^32 + float64(s & 0xffffffff): the product is
// exact, so one rounding whether or not the two are fused.
__device__ __forceinline__ double to_double(long long s) {
    const double hi = (double)(int)(s >> 32);
    const double lo = (double)(unsigned)(s & 0xFFFFFFFFll);
    return hi * 4294967296.0 + lo;
}

// Order-preserving map of fp32 to uint32 (and back), for atomic min / max.
__device__ __forceinline__ uint32_t float_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Candidate search.  A centre's window holds a sample when |p_d - c_d| <=
// C_d on every axis (Section 3.2.2).  A centre may drift any distance from
// its seed cell, so no fixed neighbourhood of seed cells is assumed: after
// each update, per axis d, every slab i (the centres with cell index i on
// axis d) records the least and greatest coordinate of its centres, and every
// seed cell j the range reach[d][j] of slabs whose [least - C, greatest + C]
// meets cell j.  A sample of cell j then tests exactly those slabs.  Rounding
// of p - c is monotone in c, so a centre that passes the window test lies in
// a slab that passes the slab test: no candidate is lost.

__device__ __forceinline__ bool slab_holds(const DevS& s, int d, int i, float p) {
    const float lo = key_float(s.slab[(0 * 4 + d) * s.kmax + i]);
    const float hi = key_float(s.slab[(1 * 4 + d) * s.kmax + i]);
    return __fsub_rn(p, hi) <= s.C[d] && __fsub_rn(p, lo) >= -s.C[d];
}

// The slabs of axis d that can hold a centre within C of p (seed cell c), as
// bits i - base.  A reach range of more than s.mask_slabs (<= 32) slabs
// (centres drifted by many cells) sets `wide`: the caller then takes
// assign_wide.
__device__ __forceinline__ unsigned axis_mask(const DevS& s, int d, int c, float p, int& base, bool& wide) {
    const int lo = s.reach[(d * s.kmax + c) * 2], hi = s.reach[(d * s.kmax + c) * 2 + 1];
    base = lo;
    if (hi < lo) return 0u;
    if (hi - lo >= s.mask_slabs) {
        wide = true;
        return 0u;
    }
    unsigned m = 0;
    for (int i = lo; i <= hi; ++i)
        if (slab_holds(s, d, i, p)) m |= 1u << (i - lo);
    return m;
}

__device__ __forceinline__ float dist2(const DevS& s, float dx, float dy, float dz, float dt) {
    const float ctd = s.cf * dt, yy = dy * dy;
    return __builtin_fmaf(ctd, ctd, __builtin_fmaf(dz, dz, __builtin_fmaf(dx, dx, yy)));
}
// A = w_v |v - v_c|
__device__ __forceinline__ float distance(const DevS& s, float A, float S) { return __builtin_fmaf(s.wd, S, A); }

// Rate centre id for the sample if its window holds it; keep the smallest D,
// ties to the lowest id.
__device__ __forceinline__ void consider(const DevS& s, int id, float px, float py, float pz, float pt, float v,
                                         bool field, float wv, float& best_d, int& best) {
    const float4 c = reinterpret_cast<const float4*>(s.cen32)[2 * id];
    const float2 cv = reinterpret_cast<const float2*>(s.cen32)[4 * id + 2];
    const float dx = __fsub_rn(px, c.x), dy = __fsub_rn(py, c.y);
    const float dz = __fsub_rn(pz, c.z), dt = __fsub_rn(pt, c.w);
    if (!(fabsf(dx) <= s.C[0] && fabsf(dy) <= s.C[1] && fabsf(dz) <= s.C[2] && fabsf(dt) <= s.C[3])) return;
    const float vc = field ? cv.y : cv.x;
    const float A = __fmul_rn(wv, fabsf(__fsub_rn(v, vc)));
    // D = A + (w_d S) rounded is >= A: a value term above the best distance
    // cannot win (nor tie), so skip the rest
    if (A > best_d) return;
    const float D = distance(s, A, __fsqrt_rn(dist2(s, dx, dy, dz, dt)));
    if (D < best_d || (D == best_d && id < best)) {
        best_d = D;
        best = id;
    }
}

// Centre with the smallest distance among the centres of the slabs in the
// masks (bit b of mx: slab bx0 + b on x, and so on); none: `prev`.
__device__ int assign_cands(const DevS& s, float px, float py, float pz, float pt, float v, bool field,
                            int prev, int bx0, int by0, int bz0, int bt0, unsigned mx, unsigned my,
                            unsigned mz, unsigned mt) {
    const float wv = field ? s.wf : s.wp;
    float best_d = INFINITY;
    int best = 0x7FFFFFFF;
    for (unsigned bt = mt; bt; bt &= bt - 1)
        for (unsigned bz = mz; bz; bz &= bz - 1)
            for (unsigned by = my; by; by &= by - 1)
                for (unsigned bx = mx; bx; bx &= bx - 1) {
                    const int ct = bt0 + __builtin_ctz(bt), cz = bz0 + __builtin_ctz(bz);
                    const int cy = by0 + __builtin_ctz(by), cx = bx0 + __builtin_ctz(bx);
                    consider(s, ((ct * s.k[2] + cz) * s.k[1] + cy) * s.k[0] + cx, px, py, pz, pt, v, field, wv,
                             best_d, best);
                }
    return best == 0x7FFFFFFF ? prev : best;
}

// The same search over reach ranges of any width (the slab test inline).
__device__ __forceinline__ int assign_wide(const DevS& s, float px, float py, float pz, float pt, float v,
                                        bool field, int prev) {
    const float p[4] = {px, py, pz, pt};
    int lo[4], hi[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int c = seed_cell(p[d], s.C[d], s.k[d]);
        lo[d] = s.reach[(d * s.kmax + c) * 2];
        hi[d] = s.reach[(d * s.kmax + c) * 2 + 1];
    }
    const float wv = field ? s.wf : s.wp;
    float best_d = INFINITY;
    int best = 0x7FFFFFFF;
    for (int ct = lo[3]; ct <= hi[3]; ++ct) {
        if (!slab_holds(s, 3, ct, pt)) continue;
        for (int cz = lo[2]; cz <= hi[2]; ++cz) {
            if (!slab_holds(s, 2, cz, pz)) continue;
            for (int cy = lo[1]; cy <= hi[1]; ++cy) {
                if (!slab_holds(s, 1, cy, py)) continue;
                for (int cx = lo[0]; cx <= hi[0]; ++cx) {
                    if (!slab_holds(s, 0, cx, px)) continue;
                    consider(s, ((ct * s.k[2] + cz) * s.k[1] + cy) * s.k[0] + cx, px, py, pz, pt, v, field, wv,
                             best_d, best);
                }
            }
        }
    }
    return best == 0x7FFFFFFF ? prev : best;
}

__device__ __forceinline__ int assign_one(const DevS& s, float px, float py, float pz, float pt, float v,
                                          bool field, int prev) {
    int b[4];
    bool wide = false;
    const unsigned mx = axis_mask(s, 0, seed_cell(px, s.C[0], s.k[0]), px, b[0], wide);
    const unsigned my = axis_mask(s, 1, seed_cell(py, s.C[1], s.k[1]), py, b[1], wide);
    const unsigned mz = axis_mask(s, 2, seed_cell(pz, s.C[2], s.k[2]), pz, b[2], wide);
    const unsigned mt = axis_mask(s, 3, seed_cell(pt, s.C[3], s.k[3]), pt, b[3], wide);
    if (wide) return assign_wide(s, px, py, pz, pt, v, field, prev);
    return assign_cands(s, px, py, pz, pt, v, field, prev, b[0], b[1], b[2], b[3], mx, my, mz, mt);
}

// Block-local sums keyed by centre id (open addressing).  A sample whose
// centre finds no free slot goes straight to the global sums.
struct Table {
    int key[kTab];
    unsigned long long acc[kTab][kSlicAcc];
};

__device__ __forceinline__ void table_init(Table& tb) {
    for (int i = threadIdx.x; i < kTab * kSlicAcc; i += blockDim.x) (&tb.acc[0][0])[i] = 0ull;
    for (int i = threadIdx.x; i < kTab; i += blockDim.x) tb.key[i] = -1;
    __syncthreads();
}

// One thread's running sums for the centre of its last samples.
struct Run {
    int id;  // -1: none
    long long q[5];
    long long n;
};

__device__ __forceinline__ void add_run(const DevS& s, Table& tb, const Run& r, bool field) {
    if (r.id < 0) return;
    const int id = r.id;
    unsigned long long* dst = nullptr;
    const unsigned h = ((unsigned)id * 2654435761u) >> 26;
    for (int k = 0; k < kTab; ++k) {
        const int slot = (h + k) & (kTab - 1);
        const int was = atomicCAS(&tb.key[slot], -1, id);
        if (was == -1 || was == id) {
            dst = tb.acc[slot];
            break;
        }
    }
    if (!dst) dst = s.acc + (size_t)id * kSlicAcc;  // table full: global (device-scope) atomics
    atomicAdd(&dst[SA_X], (unsigned long long)r.q[0]);
    atomicAdd(&dst[SA_Y], (unsigned long long)r.q[1]);
    atomicAdd(&dst[SA_Z], (unsigned long long)r.q[2]);
    atomicAdd(&dst[SA_T], (unsigned long long)r.q[3]);
    atomicAdd(&dst[field ? SA_F : SA_P], (unsigned long long)r.q[4]);
    atomicAdd(&dst[field ? SA_NF : SA_NP], (unsigned long long)r.n);
}

// Add one sample to the thread's run; a sample of another centre first adds
// the run to the block's sums.
__device__ __forceinline__ void run_sample(const DevS& s, Table& tb, Run& r, int id, const long long* q,
                                           bool field) {
    if (id != r.id) {
        add_run(s, tb, r, field);
        r.id = id;
        r.n = 0;
        for (int k = 0; k < 5; ++k) r.q[k] = 0;
    }
    for (int k = 0; k < 5; ++k) r.q[k] += q[k];
    ++r.n;
}

// A centre's sums, in the block's copy of them: with few centres every block adds
// to the same few lines, and an address takes 11 ns per device atomic.
__device__ __forceinline__ unsigned long long* centre_sums(const DevS& s, int id) {
    return s.acc + ((size_t)(blockIdx.x & (s.copies - 1)) * s.K + id) * kSlicAcc;
}

// One sample straight to its centre's sums.
__device__ __forceinline__ void add_sample(const DevS& s, int id, const int* q, bool field) {
    unsigned long long* a = centre_sums(s, id);
    for (int k = 0; k < 4; ++k) atomicAdd(&a[SA_X + k], (unsigned long long)(long long)q[k]);
    atomicAdd(&a[field ? SA_F : SA_P], (unsigned long long)(long long)q[4]);
    atomicAdd(&a[field ? SA_NF : SA_NP], 1ull);
}

__device__ __forceinline__ void table_flush(const DevS& s, Table& tb) {
    __syncthreads();
    for (int i = threadIdx.x; i < kTab * kSlicAcc; i += blockDim.x) {
        const int slot = i / kSlicAcc, a = i % kSlicAcc;
        const int id = tb.key[slot];
        const unsigned long long v = tb.acc[slot][a];
        if (id >= 0 && v) atomicAdd(&centre_sums(s, id)[a], v);
    }
}

// ---- passes over boxes of samples ------------------------------------------

// Centres a box's list holds: location, (value of the box's sample type, id).
struct Cands {
    float4 c[kCand];
    float2 v[kCand];
    uint16_t ax[4][kAxis];  // slabs met, per axis
    int nax[4];
    int n;
    float box[4][8];        // per wave: least and greatest x, y, z, t of its samples
};

template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    const int b = __float_as_int(x);
    return __int_as_float(__builtin_amdgcn_update_dpp(b, b, CTRL, 0xF, 0xF, false));
}
// Greatest value of the wave (uniform): shifts inside the rows of 16 lanes, then
// the rows' last lanes broadcast onwards; lane 63 has seen every lane.
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp_move<0x111>(x));
    x = fmaxf(x, dpp_move<0x112>(x));
    x = fmaxf(x, dpp_move<0x114>(x));
    x = fmaxf(x, dpp_move<0x118>(x));
    x = fmaxf(x, dpp_move<0x142>(x));
    x = fmaxf(x, dpp_move<0x143>(x));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ float wave_min(float x) { return -wave_max(-x); }

// Least and greatest |fl(p - c)| over p in [lo, hi]: rounding is monotone in
// p, so they are taken at the ends (or 0 between them).
struct Span {
    float least, most;
};
__device__ __forceinline__ Span span(float lo, float hi, float c) {
    const float a = __fsub_rn(lo, c), b = __fsub_rn(hi, c);
    return {fmaxf(0.0f, fmaxf(a, -b)), fmaxf(-a, b)};
}

// The centres whose window meets the box [lo, hi], into L (any order).  Wave d
// finds the slabs of axis d that can hold one; the block then tests the centres
// of their combinations.  Returns the number, or -1 when the list would not
// fit.  Every thread of the block calls it.
template <bool FIELD>
__device__ int list_cands(const DevS& s, Cands& L, const float* lo, const float* hi) {
    const int lane = threadIdx.x & 63, d = threadIdx.x >> 6;
    if (threadIdx.x == 0) L.n = 0;
    int n = 0;
    for (int i0 = 0; i0 < s.k[d]; i0 += 64) {
        const int i = i0 + lane;
        bool ok = false;
        if (i < s.k[d]) {
            const float sl = key_float(s.slab[(0 * 4 + d) * s.kmax + i]);
            const float sh = key_float(s.slab[(1 * 4 + d) * s.kmax + i]);
            ok = __fsub_rn(lo[d], sh) <= s.C[d] && __fsub_rn(hi[d], sl) >= -s.C[d];
        }
        const unsigned long long m = __ballot(ok);
        const int at = n + __popcll(m & ((1ull << lane) - 1));
        if (ok && at < kAxis) L.ax[d][at] = (uint16_t)i;
        n += __popcll(m);
    }
    if (lane == 0) L.nax[d] = n;
    __syncthreads();
    const int n0 = L.nax[0], n1 = L.nax[1], n2 = L.nax[2], n3 = L.nax[3];
    if (n0 > kAxis || n1 > kAxis || n2 > kAxis || n3 > kAxis || n0 * n1 * n2 * n3 > kRaw) return -1;
    for (unsigned r = threadIdx.x; r < (unsigned)(n0 * n1 * n2 * n3); r += kBlock) {
        unsigned q = r;
        const int cx = L.ax[0][q % n0];
        q /= n0;
        const int cy = L.ax[1][q % n1];
        q /= n1;
        const int cz = L.ax[2][q % n2], ct = L.ax[3][q / n2];
        const int id = ((ct * s.k[2] + cz) * s.k[1] + cy) * s.k[0] + cx;
        const float4 c = reinterpret_cast<const float4*>(s.cen32)[2 * id];
        const float2 cv = reinterpret_cast<const float2*>(s.cen32)[4 * id + 2];
        if (span(lo[0], hi[0], c.x).least <= s.C[0] && span(lo[1], hi[1], c.y).least <= s.C[1] &&
            span(lo[2], hi[2], c.z).least <= s.C[2] && span(lo[3], hi[3], c.w).least <= s.C[3]) {
            const int at = atomicAdd(&L.n, 1);
            if (at < kCand) {
                L.c[at] = c;
                L.v[at] = make_float2(FIELD ? cv.y : cv.x, __int_as_float(id));
            }
        }
    }
    __syncthreads();
    return L.n > kCand ? -1 : L.n;
}

// The seed cells of the box as its list (their ids); -1 when they would not
// fit.  first / num: the cells of the box per axis.
__device__ int list_cells(const DevS& s, Cands& L, const float* lo, const float* hi, int* first, int* num) {
    int64_t n = 1;
    for (int d = 0; d < 4; ++d) {
        first[d] = seed_cell(lo[d], s.C[d], s.k[d]);
        num[d] = seed_cell(hi[d], s.C[d], s.k[d]) - first[d] + 1;
        n *= num[d];
    }
    if (n > kCand) return -1;
    for (int i = threadIdx.x; i < (int)n; i += kBlock) {
        int q = i;
        const int cx = first[0] + q % num[0];
        q /= num[0];
        const int cy = first[1] + q % num[1];
        q /= num[1];
        const int cz = first[2] + q % num[2], ct = first[3] + q / num[2];
        L.v[i].y = __int_as_float(((ct * s.k[2] + cz) * s.k[1] + cy) * s.k[0] + cx);
    }
    __syncthreads();
    return (int)n;
}

// Of the n listed centres, those that can win for a sample in the wave's box
// [lo, hi] with a value in [vlo, vhi], as bits: `whole` the ones whose windows
// hold the whole box, `part` the others.  The distance's operations are monotone
// in |p - c| and |v - v_c|, so evaluating them, rounding and all, at the least and
// greatest of these bounds every sample's distance (the margin of 2^-20 covers the
// square root's last place); a centre whose lower bound exceeds the upper bound of
// one whose window holds the whole box loses for every sample.
struct Kept {
    unsigned long long whole[kCand / 64], part[kCand / 64];
};
__device__ __forceinline__ void keep_cands(const DevS& s, const Cands& L, int n, const float* lo, const float* hi,
                                           float vlo, float vhi, float wv, Kept& keep) {
    float lb[kCand / 64], best = INFINITY;
    bool meets[kCand / 64], covers[kCand / 64];
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int r = 0; r < kCand / 64; ++r) {
        meets[r] = covers[r] = false;
        lb[r] = 0.0f;
        if (r * 64 >= n) continue;  // wave-uniform
        const int i = min(r * 64 + lane, n - 1);
        const float4 c = L.c[i];
        const Span x = span(lo[0], hi[0], c.x), y = span(lo[1], hi[1], c.y);
        const Span z = span(lo[2], hi[2], c.z), t = span(lo[3], hi[3], c.w);
        const Span v = span(vlo, vhi, L.v[i].x);
        meets[r] = r * 64 + lane < n && x.least <= s.C[0] && y.least <= s.C[1] && z.least <= s.C[2] &&
                   t.least <= s.C[3];
        lb[r] = distance(s, wv * v.least, __builtin_amdgcn_sqrtf(dist2(s, x.least, y.least, z.least, t.least)));
        covers[r] = meets[r] && x.most <= s.C[0] && y.most <= s.C[1] && z.most <= s.C[2] && t.most <= s.C[3];
        const float ub = distance(s, wv * v.most, __builtin_amdgcn_sqrtf(dist2(s, x.most, y.most, z.most, t.most)));
        if (covers[r]) best = fminf(best, ub);
    }
    best = wave_min(best);
    best += best * 0x1p-20f + s.tie;
#pragma unroll
    for (int r = 0; r < kCand / 64; ++r) {
        const bool k = meets[r] && !(lb[r] > best);
        keep.whole[r] = r * 64 < n ? __ballot(k && covers[r]) : 0ull;
        keep.part[r] = r * 64 < n ? __ballot(k && !covers[r]) : 0ull;
    }
}

// fn(i) for each set bit's list index i (wave-uniform).
template <typename Fn>
__device__ __forceinline__ void each_kept(const unsigned long long* bits, int n, Fn&& fn) {
#pragma unroll
    for (int r = 0; r < kCand / 64; ++r) {
        if (r * 64 >= n) break;
        for (unsigned long long m = bits[r]; m; m &= m - 1)
            fn(__builtin_amdgcn_readfirstlane(r * 64 + __builtin_ctzll(m)));
    }
}

// The list index of the best of the kept centres for each of the lane's
// samples (-1: no window holds it).  Only where the two smallest distances are
// equal (or there are none) are the centres rated again, ties to the lowest id;
// s.tie covers the square root's scaling of denormals, which the first rating
// leaves out.
template <int N>
__device__ __forceinline__ void rate_samples(const DevS& s, const Cands& L, const Kept& keep, int n, const float* px,
                                             const float* py, const float* pz, const float* pt, const float* v,
                                             const bool* live, float wv, int* win) {
    float d1[N], d2[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        d1[j] = d2[j] = INFINITY;
        win[j] = -1;
    }
    auto rate = [&](int i, bool test) {
        const float4 c = L.c[i];
        const float vc = L.v[i].x;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float dx = px[j] - c.x, dy = py[j] - c.y, dz = pz[j] - c.z, dt = pt[j] - c.w;
            const float S = __builtin_amdgcn_sqrtf(dist2(s, dx, dy, dz, dt));
            float D = distance(s, wv * fabsf(v[j] - vc), S);
            if (test && !(fabsf(dx) <= s.C[0] && fabsf(dy) <= s.C[1] && fabsf(dz) <= s.C[2] && fabsf(dt) <= s.C[3]))
                D = INFINITY;
            if (D < d1[j]) win[j] = i;
            d2[j] = __builtin_amdgcn_fmed3f(d1[j], d2[j], D);
            d1[j] = fminf(d1[j], D);
        }
    };
    each_kept(keep.whole, n, [&](int i) { rate(i, false); });
    each_kept(keep.part, n, [&](int i) { rate(i, true); });
    bool again = false;
#pragma unroll
    for (int j = 0; j < N; ++j) again |= live[j] && !(d2[j] - d1[j] > s.tie);  // none in a window: NaN
    if (__ballot(again) == 0) return;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const bool close = live[j] && !(d2[j] - d1[j] > s.tie);
        float best_d = INFINITY;
        int best = 0x7FFFFFFF, at = -1;
        auto exact = [&](int i) {
            const float4 c = L.c[i];
            const int id = __float_as_int(L.v[i].y);
            const float dx = px[j] - c.x, dy = py[j] - c.y, dz = pz[j] - c.z, dt = pt[j] - c.w;
            if (!(fabsf(dx) <= s.C[0] && fabsf(dy) <= s.C[1] && fabsf(dz) <= s.C[2] && fabsf(dt) <= s.C[3])) return;
            const float D = distance(s, wv * fabsf(v[j] - L.v[i].x), __fsqrt_rn(dist2(s, dx, dy, dz, dt)));
            if (D < best_d || (D == best_d && id < best)) {
                best_d = D;
                best = id;
                at = i;
            }
        };
        each_kept(keep.whole, n, exact);
        each_kept(keep.part, n, exact);
        if (close) win[j] = at;
    }
}

// Box shape of the field pass, as logarithms: a lane takes four samples along
// x, a wave 8 x 2^ly x 2^lz x 2^lt, a block 2^wx waves along x and the others
// along y, each 2^(iy + iz + it) wave boxes (at most 4,096 samples in all).
struct FieldBox {
    int ly, lz, lt, wx, iy, iz, it;
    int nx, ny, nz, nt;  // boxes per axis
    int vec;             // rows are whole 16-byte vectors
    __host__ __device__ int ex() const { return 8 << wx; }
    __host__ __device__ int ey() const { return 1 << (ly + 2 - wx + iy); }
    __host__ __device__ int ez() const { return 1 << (lz + iz); }
    __host__ __device__ int et() const { return 1 << (lt + it); }
};

// A lane's place in its block's box: x, and y, z, t in each of the wave boxes.
struct FieldLane {
    int x, y, z, t, sy, steps;
    __device__ explicit FieldLane(const FieldBox& b) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        x = (wave & ((1 << b.wx) - 1)) * 8 + (lane & 1) * 4;
        y = ((wave >> b.wx) << b.ly) + ((lane >> 1) & ((1 << b.ly) - 1));
        z = (lane >> (1 + b.ly)) & ((1 << b.lz) - 1);
        t = lane >> (1 + b.ly + b.lz);
        sy = 1 << (b.ly + 2 - b.wx);  // y extent of one step
        steps = 1 << (b.iy + b.iz + b.it);
    }
    // origin of step k
    __device__ void step(const FieldBox& b, int k, int& ky, int& kz, int& kt) const {
        ky = (k & ((1 << b.iy) - 1)) * sy;
        kz = ((k >> b.iy) & ((1 << b.iz) - 1)) << b.lz;
        kt = (k >> (b.iy + b.iz)) << b.lt;
    }
    __device__ void place(const FieldBox& b, int k, int& py, int& pz, int& pt) const {
        step(b, k, py, pz, pt);
        py += y;
        pz += z;
        pt += t;
    }
};

// A block's sums of field samples per listed centre, in box coordinates packed
// into two words: n | x << 13 | y << 30 | t << 47 and value + (z << 44).  At most
// 4,096 samples, x and y below 32, z and t below 16 keep each field in its bits;
// the value (44 bits, signed) borrows from z and is taken out first.
struct FieldRun {
    int at;  // list index (-1: none)
    unsigned n, x, y, z, t;
    long long v;
};

// Note box e (field boxes, then point blocks) for the search sample by sample.
__device__ __forceinline__ void note_box(const DevS& s, uint32_t e) {
    if (threadIdx.x == 0) s.over[1 + atomicAdd(&s.over[0], 1u)] = e;
}

// Field samples, one box of FieldBox shape per block.  ASSIGN 0: labels from
// the seed cells.  Bound by the candidates' arithmetic: 4.9 ms for 1.07e9
// samples and 16,384 centres (256^3 x 64, 4 B read and 4 B written per sample),
// where testing the slab combinations sample by sample took 66 ms.
template <int ASSIGN>
__device__ __forceinline__ void field_pass(const DevS& s, const FieldBox& b, uint32_t box, Cands& L,
                                           unsigned long long (*acc)[2]) {
    const int wave = threadIdx.x >> 6;
    uint32_t r = box;
    const int x0 = (int)(r % b.nx) * b.ex();
    r /= b.nx;
    const int y0 = (int)(r % b.ny) * b.ey();
    r /= b.ny;
    const int z0 = (int)(r % b.nz) * b.ez(), t0 = (int)(r / b.nz) * b.et();
    const FieldLane at(b);
    const int lx = at.x, ly = at.y, lz = at.z, lt = at.t;
    const float lo[4] = {(float)x0 + 0.5f, (float)y0 + 0.5f, (float)z0 + 0.5f, (float)t0};
    const float hi[4] = {(float)min(x0 + b.ex(), s.X) - 0.5f, (float)min(y0 + b.ey(), s.Y) - 0.5f,
                         (float)min(z0 + b.ez(), s.Z) - 0.5f, (float)min(t0 + b.et(), s.T) - 1.0f};
    // four samples of the row at (x, y, z, t): values; which exist and are finite
    auto load = [&](size_t i, bool row, float* v, bool* in, bool* live) {
        const int x = x0 + lx;
        if (row && b.vec && x < s.X) {
            const float4 f = *reinterpret_cast<const float4*>(s.field + i);
            v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            in[j] = row && x + j < s.X;
            if (!in[j]) v[j] = 0.0f;
            else if (!b.vec) v[j] = s.field[i + j];
            live[j] = in[j] && isfinite(v[j]);
            if (live[j] && !(fabsf(v[j]) < kMaxAbs)) s.counters[SC_RANGE] = 1u;
        }
    };

    int n, first[4], num[4];
    if (ASSIGN) n = s.boxes ? list_cands<true>(s, L, lo, hi) : -1;
    else n = list_cells(s, L, lo, hi, first, num);
    if (n < 0) {  // block-uniform
        note_box(s, box);
        return;
    }
    for (int i = threadIdx.x; i < n; i += kBlock) acc[i][0] = acc[i][1] = 0ull;
    __syncthreads();
    FieldRun run{-1, 0, 0, 0, 0, 0, 0};
    auto flush = [&]() {
        if (run.at < 0) return;
        atomicAdd(&acc[run.at][0], (unsigned long long)run.n | ((unsigned long long)run.x << 13) |
                                             ((unsigned long long)run.y << 30) | ((unsigned long long)run.t << 47));
        atomicAdd(&acc[run.at][1], (unsigned long long)run.v + ((unsigned long long)run.z << 44));
    };
    for (int k = 0; k < at.steps; ++k) {
        int ky, kz, kt;
        at.step(b, k, ky, kz, kt);
        const int y = y0 + ky + ly, z = z0 + kz + lz, t = t0 + kt + lt;
        const bool row = y < s.Y && z < s.Z && t < s.T;
        const size_t i = (((size_t)t * s.Z + z) * s.Y + y) * s.X + x0 + lx;
        float v[4];
        bool in[4], live[4];
        load(i, row, v, in, live);
        const float px[4] = {(float)(x0 + lx) + 0.5f, (float)(x0 + lx + 1) + 0.5f, (float)(x0 + lx + 2) + 0.5f,
                             (float)(x0 + lx + 3) + 0.5f};
        const float fy = (float)y + 0.5f, fz = (float)z + 0.5f, ft = (float)t;
        int win[4];
        if (ASSIGN) {
            float vlo = INFINITY, vhi = -INFINITY;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (live[j]) {
                    vlo = fminf(vlo, v[j]);
                    vhi = fmaxf(vhi, v[j]);
                }
            vlo = wave_min(vlo);
            vhi = wave_max(vhi);
            // the wave box, cut to the grid (empty only where no sample is live)
            const int wx = x0 + (wave & ((1 << b.wx) - 1)) * 8, wy = y0 + ky + ((wave >> b.wx) << b.ly);
            const int wz = z0 + kz, wt = t0 + kt;
            const float wlo[4] = {(float)wx + 0.5f, (float)wy + 0.5f, (float)wz + 0.5f, (float)wt};
            const float whi[4] = {(float)min(wx + 8, s.X) - 0.5f, (float)min(wy + (1 << b.ly), s.Y) - 0.5f,
                                  (float)min(wz + (1 << b.lz), s.Z) - 0.5f, (float)min(wt + (1 << b.lt), s.T) - 1.0f};
#pragma unroll
            for (int j = 0; j < 4; ++j) win[j] = -1;
            if (vlo <= vhi) {  // wave-uniform: some sample is live
                Kept keep;
                keep_cands(s, L, n, wlo, whi, vlo, vhi, s.wf, keep);
                const float py[4] = {fy, fy, fy, fy}, pz[4] = {fz, fz, fz, fz}, pt[4] = {ft, ft, ft, ft};
                rate_samples<4>(s, L, keep, n, px, py, pz, pt, v, live, s.wf, win);
            }
        } else {
            const int c = ((seed_cell(ft, s.C[3], s.k[3]) - first[3]) * num[2] +
                           (seed_cell(fz, s.C[2], s.k[2]) - first[2])) * num[1] +
                          (seed_cell(fy, s.C[1], s.k[1]) - first[1]);
#pragma unroll
            for (int j = 0; j < 4; ++j) win[j] = c * num[0] + seed_cell(px[j], s.C[0], s.k[0]) - first[0];
        }
        int id[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            id[j] = -1;
            if (!live[j]) continue;
            if (win[j] < 0) {  // no window holds it: it keeps its centre, listed or not
                id[j] = s.labels[i + j];
                const int q[5] = {quantise(px[j]), quantise(fy), quantise(fz), t << 20, quantise(v[j])};
                add_sample(s, id[j], q, true);
                continue;
            }
            id[j] = __float_as_int(L.v[win[j]].y);
            if (win[j] != run.at) {
                flush();
                run = FieldRun{win[j], 0, 0, 0, 0, 0, 0};
            }
            run.n += 1;
            run.x += lx + j;
            run.y += ky + ly;
            run.z += kz + lz;
            run.t += kt + lt;
            run.v += quantise(v[j]);
        }
        if (b.vec && in[0]) {
            *reinterpret_cast<int4*>(s.labels + i) = make_int4(id[0], id[1], id[2], id[3]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (in[j]) s.labels[i + j] = id[j];
        }
    }
    flush();
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kBlock) {
        const unsigned long long a = acc[i][0], w = acc[i][1];
        const long long cnt = (long long)(a & 0x1FFF);
        if (!cnt) continue;
        const long long sx = (long long)((a >> 13) & 0x1FFFF), sy2 = (long long)((a >> 30) & 0x1FFFF);
        const long long st = (long long)(a >> 47);
        const long long sv = (long long)(w << 20) >> 20;  // the low 44 bits, signed
        const long long sz = (long long)(w - (unsigned long long)sv) >> 44;
        unsigned long long* o = centre_sums(s, __float_as_int(L.v[i].y));
        // q(x0 + x + 0.5) = (2 (x0 + x) + 1) 2^19
        atomicAdd(&o[SA_X], (unsigned long long)((2 * sx + (2 * x0 + 1) * cnt) << 19));
        atomicAdd(&o[SA_Y], (unsigned long long)((2 * sy2 + (2 * y0 + 1) * cnt) << 19));
        atomicAdd(&o[SA_Z], (unsigned long long)((2 * sz + (2 * z0 + 1) * cnt) << 19));
        atomicAdd(&o[SA_T], (unsigned long long)((st + t0 * cnt) << 20));
        atomicAdd(&o[SA_F], (unsigned long long)sv);
        atomicAdd(&o[SA_NF], (unsigned long long)cnt);
    }
}

// A block's sums of point samples per listed centre: x, y, z, value, and
// t | n << 48 (1,024 samples with 0 <= t < 2^31 keep t below 2^41).
struct PointRun {
    int at;
    unsigned n;
    long long q[5];
};

// Point samples in visiting order (particle-steps sorted by the sub-box holding
// them, so that a wave's are close together, with positions, times and values
// copied in that order): block b takes positions [b * 1024, (b + 1) * 1024),
// 4 consecutive ones per thread.  Their labels follow the field's, in the
// same order.  Bound like the field pass: 4.4 ms for 2.7e8 points and 16,384
// centres, 24 ms sample by sample.
template <int ASSIGN, int N>
__device__ __forceinline__ void point_pass(const DevS& s, uint32_t nfield, uint32_t blk, Cands& L,
                                           unsigned long long (*acc)[5]) {
    const int wave = threadIdx.x >> 6;
    const uint64_t V = (uint64_t)s.X * s.Y * s.Z * s.T;
    const uint64_t Q = (uint64_t)s.Tp * s.P;
    const uint64_t base = ((uint64_t)blk * kBlock + threadIdx.x) * N;
    int32_t* lab = s.labels + V + base;
    float px[N], py[N], pz[N], pt[N], v[N];
    bool in[N], live[N];
    float lo[4] = {INFINITY, INFINITY, INFINITY, INFINITY}, hi[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    float vlo = INFINITY, vhi = -INFINITY;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        in[j] = base + j < Q;
        const float4 pp = in[j] ? s.spos[base + j] : make_float4(0.f, 0.f, 0.f, 0.f);
        v[j] = in[j] ? s.sattr[base + j] : 0.0f;
        px[j] = pp.x; py[j] = pp.y; pz[j] = pp.z; pt[j] = pp.w;
        live[j] = in[j] && isfinite(v[j]) && isfinite(pp.x) && isfinite(pp.y) && isfinite(pp.z);
        if (!live[j]) continue;
        if (!(fabsf(v[j]) < kMaxAbs && fabsf(pp.x) < kMaxAbs && fabsf(pp.y) < kMaxAbs && fabsf(pp.z) < kMaxAbs))
            s.counters[SC_RANGE] = 1u;
        const float p[4] = {pp.x, pp.y, pp.z, pp.w};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            lo[d] = fminf(lo[d], p[d]);
            hi[d] = fmaxf(hi[d], p[d]);
        }
        vlo = fminf(vlo, v[j]);
        vhi = fmaxf(vhi, v[j]);
    }
    vlo = wave_min(vlo);
    vhi = wave_max(vhi);
    float blo[4], bhi[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        lo[d] = wave_min(lo[d]);
        hi[d] = wave_max(hi[d]);
        if ((threadIdx.x & 63) == 0) {
            L.box[wave][d] = lo[d];
            L.box[wave][4 + d] = hi[d];
        }
    }
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        float a = INFINITY, c = -INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            a = fminf(a, L.box[w][d]);
            c = fmaxf(c, L.box[w][4 + d]);
        }
        // no live sample in the block: any box will do
        blo[d] = a <= c ? a : 0.0f;
        bhi[d] = a <= c ? c : 0.0f;
    }

    int n, first[4], num[4];
    if (ASSIGN) n = s.boxes ? list_cands<false>(s, L, blo, bhi) : -1;
    else n = list_cells(s, L, blo, bhi, first, num);
    if (n < 0) {  // block-uniform
        note_box(s, nfield + blk);
        return;
    }
    for (int i = threadIdx.x; i < n * 5; i += kBlock) (&acc[0][0])[i] = 0ull;
    __syncthreads();
    int win[N];
#pragma unroll
    for (int j = 0; j < N; ++j) win[j] = -1;
    if (ASSIGN) {
        if (vlo <= vhi) {  // wave-uniform: some sample is live
            Kept keep;
            keep_cands(s, L, n, lo, hi, vlo, vhi, s.wp, keep);
            rate_samples<N>(s, L, keep, n, px, py, pz, pt, v, live, s.wp, win);
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (live[j])
                win[j] = (((seed_cell(pt[j], s.C[3], s.k[3]) - first[3]) * num[2] +
                           (seed_cell(pz[j], s.C[2], s.k[2]) - first[2])) * num[1] +
                          (seed_cell(py[j], s.C[1], s.k[1]) - first[1])) * num[0] +
                         (seed_cell(px[j], s.C[0], s.k[0]) - first[0]);
    }
    PointRun run{-1, 0, {0, 0, 0, 0, 0}};
    auto flush = [&]() {
        if (run.at < 0) return;
        unsigned long long* a = acc[run.at];
        atomicAdd(&a[0], (unsigned long long)run.q[0]);
        atomicAdd(&a[1], (unsigned long long)run.q[1]);
        atomicAdd(&a[2], (unsigned long long)run.q[2]);
        atomicAdd(&a[3], (unsigned long long)run.q[3] + ((unsigned long long)run.n << 48));
        atomicAdd(&a[4], (unsigned long long)run.q[4]);
    };
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (!in[j]) continue;
        if (!live[j]) {
            lab[j] = -1;
            continue;
        }
        const int q[5] = {quantise(px[j]), quantise(py[j]), quantise(pz[j]), quantise(pt[j]), quantise(v[j])};
        if (win[j] < 0) {  // no window holds it: it keeps its centre, listed or not
            add_sample(s, lab[j], q, false);
            continue;
        }
        lab[j] = __float_as_int(L.v[win[j]].y);
        if (win[j] != run.at) {
            flush();
            run = PointRun{win[j], 0, {0, 0, 0, 0, 0}};
        }
        run.n += 1;
#pragma unroll
        for (int e = 0; e < 5; ++e) run.q[e] += q[e];
    }
    flush();
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kBlock) {
        const unsigned long long* a = acc[i];
        const unsigned long long cnt = a[3] >> 48;
        if (!cnt) continue;
        unsigned long long* o = centre_sums(s, __float_as_int(L.v[i].y));
        atomicAdd(&o[SA_X], a[0]);
        atomicAdd(&o[SA_Y], a[1]);
        atomicAdd(&o[SA_Z], a[2]);
        atomicAdd(&o[SA_T], a[3] & 0xFFFFFFFFFFFFull);
        atomicAdd(&o[SA_P], a[4]);
        atomicAdd(&o[SA_NP], cnt);
    }
}

template <int ASSIGN>
__global__ __launch_bounds__(kBlock) void k_slic_field(DevS s, FieldBox b) {
    __shared__ Cands L;
    __shared__ unsigned long long acc[kCand][2];
    if (s.counters[SC_DONE]) return;
    field_pass<ASSIGN>(s, b, blockIdx.x, L, acc);
}

template <int ASSIGN, int N>
__global__ __launch_bounds__(kBlock) void k_slic_points(DevS s, uint32_t nfield) {
    __shared__ Cands L;
    __shared__ unsigned long long acc[kCand][5];
    if (s.counters[SC_DONE]) return;
    point_pass<ASSIGN, N>(s, nfield, blockIdx.x, L, acc);
}

// Both passes in one launch, one point per thread, where neither fills the GPU
// (a block's chain of loads, about 15 us, is what an iteration of 32^3 x 8 then
// waits for: once instead of twice).
template <int ASSIGN>
__global__ __launch_bounds__(kBlock) void k_slic_both(DevS s, FieldBox b, uint32_t nfield) {
    __shared__ Cands L;
    __shared__ unsigned long long acc[kCand][5];
    if (s.counters[SC_DONE]) return;
    if (blockIdx.x < nfield)
        field_pass<ASSIGN>(s, b, blockIdx.x, L, reinterpret_cast<unsigned long long(*)[2]>(&acc[0][0]));
    else
        point_pass<ASSIGN, 1>(s, nfield, blockIdx.x - nfield, L, acc);
}

// The boxes whose list did not fit, sample by sample through the slabs' reach
// ranges.  npoint: points per noted block.  A kernel of its own, so that its
// registers do not cost the passes their occupancy: inside them it held them at
// 119 and 101 registers, four waves per SIMD, and 9.8 and 7.8 ms instead of 4.9
// and 4.4 ms at 256^3 x 64.
template <int ASSIGN>
__global__ __launch_bounds__(kBlock) void k_slic_rest(DevS s, FieldBox b, uint32_t nfield, uint32_t npoint) {
    __shared__ Table tb;
    if (s.counters[SC_DONE]) return;
    const uint32_t count = s.over[0];
    const uint64_t V = (uint64_t)s.X * s.Y * s.Z * s.T, Q = (uint64_t)s.Tp * s.P;
    for (uint32_t e = blockIdx.x; e < count; e += gridDim.x) {
        const uint32_t box = s.over[1 + e];
        const bool field = box < nfield;
        __syncthreads();
        table_init(tb);
        Run run;
        run.id = -1;
        int x0 = 0, y0 = 0, z0 = 0, t0 = 0;
        if (field) {
            uint32_t r = box;
            x0 = (int)(r % b.nx) * b.ex();
            r /= b.nx;
            y0 = (int)(r % b.ny) * b.ey();
            r /= b.ny;
            z0 = (int)(r % b.nz) * b.ez();
            t0 = (int)(r / b.nz) * b.et();
        }
        // four consecutive samples per thread (along x for the field)
        const uint32_t n = field ? (uint32_t)(b.ex() * b.ey() * b.ez() * b.et()) : npoint;
        for (uint32_t i0 = threadIdx.x * 4; i0 < n; i0 += kBlock * 4) {
            for (int j = 0; j < 4; ++j) {
                float px, py, pz, pt, v;
                size_t at;  // label
                if (field) {
                    uint32_t r = i0 + j;
                    const int x = x0 + (int)(r % b.ex());
                    r /= b.ex();
                    const int y = y0 + (int)(r % b.ey());
                    r /= b.ey();
                    const int z = z0 + (int)(r % b.ez()), t = t0 + (int)(r / b.ez());
                    if (x >= s.X || y >= s.Y || z >= s.Z || t >= s.T) continue;
                    at = (((size_t)t * s.Z + z) * s.Y + y) * s.X + x;
                    px = (float)x + 0.5f;
                    py = (float)y + 0.5f;
                    pz = (float)z + 0.5f;
                    pt = (float)t;
                    v = s.field[at];
                } else {
                    const uint64_t o = (uint64_t)(box - nfield) * npoint + i0 + j;
                    if (i0 + j >= n || o >= Q) continue;
                    const float4 pp = s.spos[o];
                    px = pp.x;
                    py = pp.y;
                    pz = pp.z;
                    pt = pp.w;
                    v = s.sattr[o];
                    at = V + o;
                }
                if (!(isfinite(v) && isfinite(px) && isfinite(py) && isfinite(pz))) {
                    s.labels[at] = -1;
                    continue;
                }
                if (!(fabsf(v) < kMaxAbs && fabsf(px) < kMaxAbs && fabsf(py) < kMaxAbs && fabsf(pz) < kMaxAbs))
                    s.counters[SC_RANGE] = 1u;
                int id;
                if (ASSIGN) {
                    id = assign_one(s, px, py, pz, pt, v, field, s.labels[at]);
                } else {
                    const int cx = seed_cell(px, s.C[0], s.k[0]), cy = seed_cell(py, s.C[1], s.k[1]);
                    const int cz = seed_cell(pz, s.C[2], s.k[2]), ct = seed_cell(pt, s.C[3], s.k[3]);
                    id = ((ct * s.k[2] + cz) * s.k[1] + cy) * s.k[0] + cx;
                }
                s.labels[at] = id;
                const long long q[5] = {quantise(px), quantise(py), quantise(pz), quantise(pt), quantise(v)};
                run_sample(s, tb, run, id, q, field);
            }
        }
        add_run(s, tb, run, field);
        table_flush(s, tb);
    }
}

// The update's slab bounds, read by the block that finishes it (written by
// other blocks' atomics: agent-scope loads, so that no stale line is read).
__device__ __forceinline__ float next_slab(const DevS& s, int i) {
    return key_float(__hip_atomic_load(&s.slab_next[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// One thread per centre.  seed: write the seed centre first (its location
// ((i + 0.5) C_d), values 0).  Then the means of the sums (a centre without
// samples, or without samples of one type, keeps the previous values), the
// convergence test against the previous centre, and the sums cleared.  A block
// gathers its centres' slab bounds in LDS first: 256 neighbouring centres share
// a few dozen slabs, and the same address takes 11 ns per device atomic (16,384
// centres: 312 us of them straight to memory, 15 us now).
//
// The last block to finish writes the reach ranges of the new slabs, clears the
// slab buffer the passes have read (the next update's), counts the iteration,
// notes a run that is done (nothing moved, a value out of range) and reports to
// the host.
constexpr int kSlabLds = 256;  // slabs per axis gathered in LDS
__global__ __launch_bounds__(256) void k_slic_update(DevS s, int seed) {
    __shared__ uint32_t s_slab[2][4][kSlabLds];
    __shared__ uint32_t s_last;
    if (s.counters[SC_DONE]) return;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool gather = s.kmax <= kSlabLds;
    for (int j = threadIdx.x; gather && j < 4 * kSlabLds; j += blockDim.x) {
        (&s_slab[0][0][0])[j] = 0xFFFFFFFFu;
        (&s_slab[1][0][0])[j] = 0u;
    }
    __syncthreads();
    bool moved = false;
    if (i < s.K) {
        double* c = s.cen + (size_t)i * 6;
        if (seed) {
            int r = i;
            const int cx = r % s.k[0];
            r /= s.k[0];
            const int cy = r % s.k[1];
            r /= s.k[1];
            const int cz = r % s.k[2];
            const int ct = r / s.k[2];
            c[0] = (double)__fmul_rn((float)cx + 0.5f, s.C[0]);
            c[1] = (double)__fmul_rn((float)cy + 0.5f, s.C[1]);
            c[2] = (double)__fmul_rn((float)cz + 0.5f, s.C[2]);
            c[3] = (double)__fmul_rn((float)ct + 0.5f, s.C[3]);
            c[4] = 0.0;
            c[5] = 0.0;
        }
        long long sum[kSlicAcc] = {};
#pragma unroll 2
        for (int q = 0; q < s.copies; ++q) {
            unsigned long long* a = s.acc + ((size_t)q * s.K + i) * kSlicAcc;
#pragma unroll
            for (int j = 0; j < kSlicAcc; ++j) {
                sum[j] += (long long)a[j];
                a[j] = 0ull;
            }
        }
#pragma unroll
        for (int j = 0; j < kSlicAcc; ++j) s.lsum[(size_t)i * kSlicAcc + j] = sum[j];  // kept for the features (Section 3.3)
        const long long nf = sum[SA_NF], np = sum[SA_NP], n = nf + np;
        double nw[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) nw[j] = c[j];
        if (n > 0)
            for (int j = 0; j < 4; ++j) nw[j] = __ddiv_rn(to_double(sum[SA_X + j]), (double)n) * kQInv;
        if (np > 0) nw[4] = __ddiv_rn(to_double(sum[SA_P]), (double)np) * kQInv;
        if (nf > 0) nw[5] = __ddiv_rn(to_double(sum[SA_F]), (double)nf) * kQInv;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            if (fabs(__dsub_rn(nw[j], c[j])) > __dmul_rn(s.eps, fabs(c[j]))) moved = true;
            c[j] = nw[j];
            s.cen32[(size_t)i * 8 + j] = (float)nw[j];
        }
        s.cnt[(size_t)i * 2] = nf;
        s.cnt[(size_t)i * 2 + 1] = np;
        // slab bounds of the new centre, on each axis (from the fp32 copy the
        // assignment compares with)
        int r = i;
        for (int d = 0; d < 4; ++d) {
            const int cell = d < 3 ? r % s.k[d] : r;
            r /= s.k[d];
            const uint32_t key = float_key((float)nw[d]);
            uint32_t* lo = gather ? &s_slab[0][d][cell] : &s.slab_next[(0 * 4 + d) * s.kmax + cell];
            uint32_t* hi = gather ? &s_slab[1][d][cell] : &s.slab_next[(1 * 4 + d) * s.kmax + cell];
            atomicMin(lo, key);
            atomicMax(hi, key);
        }
    }
    const unsigned long long m = __ballot(moved);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(&s.counters[SC_MOVED], (unsigned)__popcll(m));
    __syncthreads();
    for (int j = threadIdx.x; gather && j < 4 * s.kmax; j += blockDim.x) {
        const int d = j / s.kmax, cell = j - d * s.kmax;
        if (s_slab[0][d][cell] > s_slab[1][d][cell]) continue;  // none of the block's centres
        atomicMin(&s.slab_next[j], s_slab[0][d][cell]);
        atomicMax(&s.slab_next[4 * s.kmax + j], s_slab[1][d][cell]);
    }
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(&s.counters[SC_TICKET], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
                 gridDim.x - 1;
    __syncthreads();
    if (!s_last) return;
    // Reach: slab i of axis d (bounds lo, hi) can hold a centre within C of any p
    // in [lo - C, hi + C], widened by C 2^-20 for the rounding of the window test's
    // difference.  Those p fall in the seed cells from floor of the lower end / C to
    // floor of the upper end / C (clamped like seed_cell), widened by 10^-3 of a
    // cell for the rounding of the division (below 2.5e-4 of a cell wherever the
    // cell index is below 4096).  Each of those cells takes i into its range.
    for (int j = threadIdx.x; j < 8 * s.kmax; j += blockDim.x) {
        s.reach[j] = (j & 1) ? -1 : 0x7FFFFFFF;
        s.slab[j] = j < 4 * s.kmax ? 0xFFFFFFFFu : 0u;
    }
    __threadfence();
    __syncthreads();
    for (int g = threadIdx.x; g < 4 * s.kmax; g += blockDim.x) {
        const int d = g / s.kmax, cell = g - d * s.kmax;
        if (cell >= s.k[d]) continue;
        const double C = s.C[d];
        const double lo = next_slab(s, g), hi = next_slab(s, 4 * s.kmax + g);
        const double w = C * (1.0 + 0x1p-20);
        const double kd = s.k[d] - 1;
        const int j0 = (int)fmin(fmax(floor((lo - w) / C - 1e-3), 0.0), kd);
        const int j1 = (int)fmin(fmax(floor((hi + w) / C + 1e-3), 0.0), kd);
        for (int j = j0; j <= j1; ++j) {
            atomicMin(&s.reach[(d * s.kmax + j) * 2], cell);
            atomicMax(&s.reach[(d * s.kmax + j) * 2 + 1], cell);
        }
    }
    if (threadIdx.x == 0) {
        const uint32_t mv =
            __hip_atomic_load(&s.counters[SC_MOVED], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t range = s.counters[SC_RANGE];
        const uint32_t iters = s.counters[SC_ITERS] + (seed ? 0u : 1u);
        s.counters[SC_ITERS] = iters;
        s.counters[SC_TICKET] = 0u;
        s.counters[SC_MOVED] = 0u;
        s.over[0] = 0u;
        const uint32_t done = range || (!seed && mv == 0u);
        if (done) s.counters[SC_DONE] = 1u;
        s.host[SC_RANGE] = range;
        s.host[SC_ITERS] = iters;
        s.host[SC_DONE] = done;
    }
}

// The start of a run: sums, counters and the first update's slab buffer cleared.
__global__ __launch_bounds__(256) void k_slic_begin(DevS s) {
    const uint64_t n = (uint64_t)s.copies * s.K * kSlicAcc;
    const uint64_t gid = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    for (uint64_t i = gid; i < n; i += (uint64_t)gridDim.x * blockDim.x) s.acc[i] = 0ull;
    if (gid < kSlicCounters) s.counters[gid] = 0u;
    if (gid == 0) s.over[0] = 0u;
    for (uint64_t i = gid; i < 8u * s.kmax; i += (uint64_t)gridDim.x * blockDim.x)
        s.slab_next[i] = i < 4u * s.kmax ? 0xFFFFFFFFu : 0u;
}

inline unsigned blocks_for(uint64_t n, uint64_t per) { return (unsigned)((n + per - 1) / per); }

// ---- cluster merging and feature statistics (Section 3.3) ------------------
//
// Centres i < j match when, per sample type, neither has samples of it or
// both do and their means differ by at most eps * max(|a|, |b|); centres
// without samples match nothing.  Features are the connected components of
// "match" (a lock-free union-find: a root is only ever linked to a smaller
// root, so every component ends rooted at its lowest centre id, whatever the
// order of the unions).  Per feature: exact means from the integer sums of
// its centres, extents and squared deviations from one pass over the samples
// keyed by centre (spatially coherent, like the clustering passes), folded
// into the features.

// Links are read with agent-scope atomic loads: a stale cached link could
// keep a compare-and-swap loop failing.
__device__ __forceinline__ int load_link(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of i, halving the path on the way (i's link moves to its grandparent:
// still an ancestor, and only a non-root's link moves, which no union
// touches).  Links strictly decrease, so the walk is at most K steps (the
// bound only guards against the impossible).
__device__ __forceinline__ int find_root(int* parent, int i, int K) {
    for (int k = 0; k <= K; ++k) {
        const int p = load_link(&parent[i]);
        if (p == i) return i;
        const int gp = load_link(&parent[p]);
        if (gp != p) __hip_atomic_store(&parent[i], gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        i = gp;
    }
    return -1;
}

__device__ bool unite(int* parent, int i, int j, int K) {
    for (int k = 0; k <= K + 1; ++k) {  // every failed swap means another union succeeded
        int a = find_root(parent, i, K), b = find_root(parent, j, K);
        if (a < 0 || b < 0) return false;
        if (a == b) return true;
        if (a > b) {
            const int t = a;
            a = b;
            b = t;
        }
        if (atomicCAS(&parent[b], b, a) == b) return true;
    }
    return false;
}

__device__ __forceinline__ bool has_samples(const DevS& s, int i) {
    return s.cnt[2 * (size_t)i] + s.cnt[2 * (size_t)i + 1] > 0;
}

__global__ __launch_bounds__(256) void k_merge_init(DevS s, DevM m) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m.K) return;
    m.parent[i] = i;
    for (int d = 0; d < 8; ++d) {
        m.cext[8 * (size_t)i + d] = d < 4 ? 0xFFFFFFFFu : 0u;
        m.fext[8 * (size_t)i + d] = d < 4 ? 0xFFFFFFFFu : 0u;
        m.fsum[8 * (size_t)i + d] = 0ull;
    }
    for (int t = 0; t < 2; ++t) {
        m.css[2 * (size_t)i + t] = 0.0;
        m.fss[2 * (size_t)i + t] = 0.0;
    }
}

// Pair tests in tiles of 256 x 256 centres, so that every block does the same
// work (K^2 / 2 tests in all): block (bx, by >= bx) compares the centres of
// tile bx, a row each, with the later centres of tile by, held in LDS.  Two
// centres match when they have the same sample types and, per type, means
// within eps of the larger magnitude (Section 3.3).  The block's matches are
// united in a union-find of the two tiles' centres in LDS, and each centre then with its
// local root in memory: at most one walk over memory per centre and block, side by side,
// instead of one after another for every match of a thread (16,384 centres: 1.5
// to 0.8 ms).  Up to kMergeSmall centres the tiles are 64 x 64 and four threads
// share a row, so that no thread walks more than 16 pairs (128 centres: 16 us, 117
// at first); with more the extra blocks only add walks.
constexpr int kMergeSmall = 4096;
__device__ __forceinline__ int lds_link(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Root of local centre i, halving the path (links strictly decrease, as above).
__device__ __forceinline__ int lds_root(int* link, int i) {
    for (;;) {
        const int p = lds_link(&link[i]);
        if (p == i) return i;
        const int gp = lds_link(&link[p]);
        if (gp != p) __hip_atomic_store(&link[i], gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        i = gp;
    }
}
template <int TILE>
__global__ __launch_bounds__(256) void k_merge_pairs(DevS s, DevM m) {
    constexpr int kShare = 256 / TILE;  // threads per row
    if (blockIdx.y < blockIdx.x) return;  // block-uniform: lower triangle
    __shared__ double sv[2][TILE];  // field mean, point mean
    __shared__ unsigned sh[TILE];   // bit 0: has field samples, bit 1: has point samples
    __shared__ int link[2 * TILE];  // tile bx, then tile by (a diagonal block uses the first half)
    const int j0 = blockIdx.y * TILE;
    const int jl = blockIdx.x == blockIdx.y ? 0 : TILE;
    if (threadIdx.x < TILE) {
        const int j = j0 + threadIdx.x;
        unsigned h = 0;
        double vf = 0.0, vp = 0.0;
        if (j < m.K) {
            h = (s.cnt[2 * (size_t)j] > 0 ? 1u : 0u) | (s.cnt[2 * (size_t)j + 1] > 0 ? 2u : 0u);
            vf = s.cen[6 * (size_t)j + 5];
            vp = s.cen[6 * (size_t)j + 4];
        }
        sh[threadIdx.x] = h;
        sv[0][threadIdx.x] = vf;
        sv[1][threadIdx.x] = vp;
        link[threadIdx.x] = threadIdx.x;
        link[TILE + threadIdx.x] = TILE + threadIdx.x;
    }
    __syncthreads();
    const int il = threadIdx.x % TILE, i = blockIdx.x * TILE + il;
    const unsigned hi = i >= m.K ? 0u : (s.cnt[2 * (size_t)i] > 0 ? 1u : 0u) | (s.cnt[2 * (size_t)i + 1] > 0 ? 2u : 0u);
    if (hi) {  // a centre without samples merges with nothing
        const double af = s.cen[6 * (size_t)i + 5], ap = s.cen[6 * (size_t)i + 4];
        const int jn = min(TILE, m.K - j0);
        int root = il;  // this centre's root when last looked up
        for (int jj = threadIdx.x / TILE; jj < jn; jj += kShare) {
            const int j = j0 + jj;
            if (j <= i || sh[jj] != hi) continue;  // a type only one has: different phenomena
            if (lds_link(&link[jl + jj]) == root) continue;  // known to be in one component already
            bool ok = true;
            if (hi & 1u) {
                const double b = sv[0][jj];
                ok = fabs(__dsub_rn(af, b)) <= __dmul_rn(m.eps, fmax(fabs(af), fabs(b)));
            }
            if (ok && (hi & 2u)) {
                const double b = sv[1][jj];
                ok = fabs(__dsub_rn(ap, b)) <= __dmul_rn(m.eps, fmax(fabs(ap), fabs(b)));
            }
            if (!ok) continue;
            for (;;) {  // every failed swap means another union succeeded
                const int a = lds_root(link, root), b = lds_root(link, jl + jj);
                root = a;
                if (a == b) break;
                const int lo = min(a, b), up = max(a, b);
                if (atomicCAS(&link[up], up, lo) == up) {
                    root = lo;
                    break;
                }
            }
        }
    }
    __syncthreads();
    for (int l = threadIdx.x; l < jl + TILE; l += 256) {
        const int r = lds_root(link, l);
        if (r == l) continue;  // (centres past K match nothing and stay roots)
        const int gl = l < TILE ? blockIdx.x * TILE + l : j0 + l - TILE;
        const int gr = r < TILE ? blockIdx.x * TILE + r : j0 + r - TILE;
        if (!unite(m.parent, gl, gr, m.K)) m.err[0] = 1u;
    }
}

__global__ __launch_bounds__(256) void k_merge_flatten(DevS s, DevM m) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m.K) return;
    int f = -1;
    if (has_samples(s, i)) {
        f = find_root(m.parent, i, m.K);
        if (f < 0) m.err[0] = 1u;
    }
    m.feat[i] = f;
}

// The lanes of a wave that hold centres of one feature combine their values
// first, so that one lane per (wave, feature) updates the feature, where at least
// kCombine lanes share it (most centres of a wave usually share one); a feature
// with fewer lanes is updated by each: combining costs about 1 us per feature
// whatever its lanes, 78 and 70 us of the two kernels when 64 centres were 64
// features.  Visits each distinct feature of the wave in turn: fn(feature, this
// lane holds it, this lane updates it, the lanes combine); F < 0: no centre.
constexpr int kCombine = 8;
template <typename Fn>
__device__ __forceinline__ void per_wave_feature(int F, Fn&& fn) {
    unsigned long long pending = __ballot(F >= 0);
    bool alone = false;
    while (pending) {  // wave-uniform
        const int leader = __ffsll((long long)pending) - 1;
        const int FL = __shfl(F, leader);
        const bool mine = F == FL;
        const unsigned long long group = __ballot(mine);
        pending &= ~group;
        if (__popcll(group) >= kCombine) fn(FL, mine, (int)__lane_id() == leader, true);
        else alone |= mine;
    }
    if (__ballot(alone)) fn(F, alone, alone, false);
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ __launch_bounds__(256) void k_feature_sums(DevS s, DevM m) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int F = i < m.K ? m.feat[i] : -1;
    unsigned long long v[kSlicAcc];
    for (int j = 0; j < kSlicAcc; ++j) v[j] = F >= 0 ? s.lsum[8 * (size_t)i + j] : 0ull;
    per_wave_feature(F, [&](int FL, bool mine, bool lead, bool combine) {
        for (int j = 0; j < kSlicAcc; ++j) {
            const unsigned long long x = combine ? wave_sum_u64(mine ? v[j] : 0ull) : v[j];
            if (lead) atomicAdd(&m.fsum[8 * (size_t)FL + j], x);
        }
    });
}

__global__ __launch_bounds__(256) void k_feature_means(DevS s, DevM m) {
    const int F = blockIdx.x * blockDim.x + threadIdx.x;
    if (F >= m.K || m.feat[F] != F) return;
    const unsigned long long* a = m.fsum + 8 * (size_t)F;
    const long long nf = (long long)a[SA_NF], np = (long long)a[SA_NP];
    m.fmean[2 * (size_t)F] = nf > 0 ? __ddiv_rn(to_double((long long)a[SA_F]), (double)nf) * kQInv : 0.0;
    m.fmean[2 * (size_t)F + 1] = np > 0 ? __ddiv_rn(to_double((long long)a[SA_P]), (double)np) * kQInv : 0.0;
}

// Block-local extents and squared deviations keyed by centre.
struct StatTable {
    int key[kTab];
    uint32_t ext[kTab][8];
    double ss[kTab];
};

struct StatRun {
    int id;
    uint32_t ext[8];
    double ss;
};

__device__ __forceinline__ void stat_init(StatTable& tb) {
    for (int i = threadIdx.x; i < kTab; i += blockDim.x) {
        tb.key[i] = -1;
        tb.ss[i] = 0.0;
        for (int d = 0; d < 8; ++d) tb.ext[i][d] = d < 4 ? 0xFFFFFFFFu : 0u;
    }
    __syncthreads();
}

__device__ __forceinline__ void stat_add(const DevM& m, StatTable& tb, const StatRun& r, int ty) {
    if (r.id < 0) return;
    uint32_t* ext = nullptr;
    double* ss = nullptr;
    const unsigned h = ((unsigned)r.id * 2654435761u) >> 26;
    for (int k = 0; k < kTab; ++k) {
        const int slot = (h + k) & (kTab - 1);
        const int was = atomicCAS(&tb.key[slot], -1, r.id);
        if (was == -1 || was == r.id) {
            ext = tb.ext[slot];
            ss = &tb.ss[slot];
            break;
        }
    }
    if (!ext) {  // table full: straight to the centre's accumulators
        ext = m.cext + 8 * (size_t)r.id;
        ss = m.css + 2 * (size_t)r.id + ty;
    }
    for (int d = 0; d < 4; ++d) {
        atomicMin(&ext[d], r.ext[d]);
        atomicMax(&ext[4 + d], r.ext[4 + d]);
    }
    atomicAdd(ss, r.ss);
}

__device__ __forceinline__ void stat_sample(const DevM& m, StatTable& tb, StatRun& r, int id, const float* c,
                                            double dev, int ty) {
    if (id != r.id) {
        stat_add(m, tb, r, ty);
        r.id = id;
        r.ss = 0.0;
        for (int d = 0; d < 4; ++d) {
            r.ext[d] = 0xFFFFFFFFu;
            r.ext[4 + d] = 0u;
        }
    }
    for (int d = 0; d < 4; ++d) {
        const uint32_t k = float_key(c[d]);
        r.ext[d] = min(r.ext[d], k);
        r.ext[4 + d] = max(r.ext[4 + d], k);
    }
    r.ss += dev * dev;
}

__device__ __forceinline__ void stat_flush(const DevM& m, StatTable& tb, int ty) {
    __syncthreads();
    for (int slot = threadIdx.x; slot < kTab; slot += blockDim.x) {
        const int id = tb.key[slot];
        if (id < 0) continue;
        for (int d = 0; d < 4; ++d) {
            atomicMin(&m.cext[8 * (size_t)id + d], tb.ext[slot][d]);
            atomicMax(&m.cext[8 * (size_t)id + 4 + d], tb.ext[slot][4 + d]);
        }
        atomicAdd(&m.css[2 * (size_t)id + ty], tb.ss[slot]);
    }
}

// Field samples, a box of FieldBox shape per block.  The extent of a centre's
// samples within the box is one word of bits, one per coordinate (x from bit 0,
// then y, z, t), so a run of samples costs an OR and an addition in LDS instead of
// eight minima and maxima, and the mean is looked up once per run: 2.6 ms for
// 1.07e9 samples (6.4 ms with consecutive samples and a table of bounds; 2.0 ms
// is what reading values and labels takes).
struct BoxTable {
    int key[kTab];
    unsigned long long bits[kTab];
    double ss[kTab];
};

// A centre's samples in a box, to its extents and squared deviations.
__device__ __forceinline__ void box_extent(const DevM& m, const FieldBox& b, int id, unsigned long long bits, double ss,
                                           int x0, int y0, int z0, int t0) {
    uint32_t* ext = m.cext + 8 * (size_t)id;
    const int o[4] = {x0, y0, z0, t0}, n[4] = {b.ex(), b.ey(), b.ez(), b.et()};
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const unsigned long long w = bits & (~0ull >> (64 - n[d]));
        bits >>= n[d];
        const float h = d < 3 ? 0.5f : 0.0f;
        atomicMin(&ext[d], float_key((float)(o[d] + __builtin_ctzll(w)) + h));
        atomicMax(&ext[4 + d], float_key((float)(o[d] + 63 - __builtin_clzll(w)) + h));
    }
    atomicAdd(&m.css[2 * (size_t)id], ss);
}

__global__ __launch_bounds__(kBlock) void k_feature_field(DevS s, DevM m, FieldBox b) {
    __shared__ BoxTable tb;
    for (int i = threadIdx.x; i < kTab; i += kBlock) {
        tb.key[i] = -1;
        tb.bits[i] = 0ull;
        tb.ss[i] = 0.0;
    }
    __syncthreads();
    uint32_t r = blockIdx.x;
    const int x0 = (int)(r % b.nx) * b.ex();
    r /= b.nx;
    const int y0 = (int)(r % b.ny) * b.ey();
    r /= b.ny;
    const int z0 = (int)(r % b.nz) * b.ez(), t0 = (int)(r / b.nz) * b.et();
    const FieldLane at(b);
    int id = -1;
    unsigned long long bits = 0;
    double ss = 0.0, mean = 0.0;
    auto flush = [&]() {
        if (id < 0) return;
        const unsigned h = ((unsigned)id * 2654435761u) >> 26;
        for (int k = 0; k < kTab; ++k) {
            const int slot = (h + k) & (kTab - 1);
            const int was = atomicCAS(&tb.key[slot], -1, id);
            if (was == -1 || was == id) {
                atomicOr(&tb.bits[slot], bits);
                atomicAdd(&tb.ss[slot], ss);
                return;
            }
        }
        box_extent(m, b, id, bits, ss, x0, y0, z0, t0);  // table full
    };
    for (int k = 0; k < at.steps; ++k) {
        int y, z, t;
        at.place(b, k, y, z, t);
        if (y0 + y >= s.Y || z0 + z >= s.Z || t0 + t >= s.T || x0 + at.x >= s.X) continue;
        const size_t i = (((size_t)(t0 + t) * s.Z + z0 + z) * s.Y + y0 + y) * s.X + x0 + at.x;
        const unsigned long long row = ((((1ull << t) << b.ez() | (1ull << z)) << b.ey()) | (1ull << y)) << b.ex();
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        int L[4] = {-1, -1, -1, -1};
        if (b.vec) {
            const float4 f = *reinterpret_cast<const float4*>(s.field + i);
            const int4 q = *reinterpret_cast<const int4*>(s.labels + i);
            v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
            L[0] = q.x; L[1] = q.y; L[2] = q.z; L[3] = q.w;
        } else {
            for (int j = 0; j < 4 && x0 + at.x + j < s.X; ++j) {
                v[j] = s.field[i + j];
                L[j] = s.labels[i + j];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (L[j] < 0) continue;
            if (L[j] != id) {
                flush();
                id = L[j];
                bits = 0;
                ss = 0.0;
                mean = m.fmean[2 * (size_t)m.feat[id]];
            }
            bits |= row | (1ull << (at.x + j));
            const double dev = (double)v[j] - mean;
            ss += dev * dev;
        }
    }
    flush();
    __syncthreads();
    for (int slot = threadIdx.x; slot < kTab; slot += kBlock)
        if (tb.key[slot] >= 0) box_extent(m, b, tb.key[slot], tb.bits[slot], tb.ss[slot], x0, y0, z0, t0);
}

// Point samples in visiting order.
__global__ __launch_bounds__(kBlock) void k_feature_points(DevS s, DevM m) {
    __shared__ StatTable tb;
    stat_init(tb);
    const uint64_t V = (uint64_t)s.X * s.Y * s.Z * s.T;
    const uint64_t N = (uint64_t)s.Tp * s.P;
    const uint64_t base = (uint64_t)blockIdx.x * (kBlock * kPer) + (uint64_t)threadIdx.x * kPer;
    StatRun run;
    run.id = -1;
    double mean = 0.0;
    for (int j = 0; j < kPer; ++j) {
        const uint64_t i = base + j;
        if (i >= N) break;
        const int L = s.labels[V + i];
        if (L < 0) continue;
        const float4 pp = s.spos[i];
        const float c[4] = {pp.x, pp.y, pp.z, pp.w};
        if (L != run.id) mean = m.fmean[2 * (size_t)m.feat[L] + 1];
        stat_sample(m, tb, run, L, c, (double)s.sattr[i] - mean, 1);
    }
    stat_add(m, tb, run, 1);
    stat_flush(m, tb, 1);
}

// Per-centre extents and squared deviations folded into their features, one
// update per (wave, feature).
__global__ __launch_bounds__(256) void k_feature_fold(DevM m) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int F = i < m.K ? m.feat[i] : -1;
    uint32_t e[8];
    double q[2];
    for (int d = 0; d < 8; ++d) e[d] = F >= 0 ? m.cext[8 * (size_t)i + d] : (d < 4 ? 0xFFFFFFFFu : 0u);
    for (int t = 0; t < 2; ++t) q[t] = F >= 0 ? m.css[2 * (size_t)i + t] : 0.0;
    per_wave_feature(F, [&](int FL, bool mine, bool lead, bool combine) {
        for (int d = 0; d < 8; ++d) {
            uint32_t x = mine ? e[d] : (d < 4 ? 0xFFFFFFFFu : 0u);
            for (int o = combine ? 32 : 0; o > 0; o >>= 1) {
                const uint32_t y = __shfl_xor(x, o);
                x = d < 4 ? min(x, y) : max(x, y);
            }
            if (lead) {
                if (d < 4) atomicMin(&m.fext[8 * (size_t)FL + d], x);
                else atomicMax(&m.fext[8 * (size_t)FL + d], x);
            }
        }
        for (int t = 0; t < 2; ++t) {
            double x = mine ? q[t] : 0.0;
            for (int o = combine ? 32 : 0; o > 0; o >>= 1) x += __shfl_xor(x, o);
            if (lead) atomicAdd(&m.fss[2 * (size_t)FL + t], x);
        }
    });
}

__global__ __launch_bounds__(256) void k_feature_write(DevM m) {
    const int F = blockIdx.x * blockDim.x + threadIdx.x;
    if (F >= m.K) return;
    double* o = m.out + (size_t)F * kFeatStats;
    for (int k = 0; k < kFeatStats; ++k) o[k] = 0.0;
    if (m.feat[F] != F) return;
    const unsigned long long* a = m.fsum + 8 * (size_t)F;
    const double nf = (double)(long long)a[SA_NF], np = (double)(long long)a[SA_NP];
    o[FS_NF] = nf;
    o[FS_NP] = np;
    o[FS_MEAN_F] = m.fmean[2 * (size_t)F];
    o[FS_MEAN_P] = m.fmean[2 * (size_t)F + 1];
    o[FS_STD_F] = nf > 0 ? sqrt(m.fss[2 * (size_t)F] / nf) : 0.0;
    o[FS_STD_P] = np > 0 ? sqrt(m.fss[2 * (size_t)F + 1] / np) : 0.0;
    for (int d = 0; d < 4; ++d) {
        o[FS_XMIN + 2 * d] = (double)key_float(m.fext[8 * (size_t)F + d]);
        o[FS_XMIN + 2 * d + 1] = (double)key_float(m.fext[8 * (size_t)F + 4 + d]);
    }
}

// ---- visiting order of the point samples (counting sort by sub-box) --------

constexpr uint32_t kSkip = 0xFFFFFFFFu;  // a padding step (t >= T): not a sample
constexpr int kScanBlocks = 1024;

// Sort key of a particle-step: the sub-box of 8 x 4 x 4 x 4 voxel-steps holding
// it, tile by tile, in an order that doubles one axis after another (y, z, x, t),
// so that 256 consecutive points fill a compact box.  Keys by tile (32 x 8 x 8 x
// BT) left a wave's points spread over the whole tile: 9.1 instead of 7.8 ms
// per point pass (as it was then) at 256^3 x 64 with 4.2 million particles.  Sub-boxes of 4 x 4 x 4
// x 2 sort 9 ms longer for the same pass.
__device__ __forceinline__ uint32_t order_key(uint32_t bin, int logBT, uint32_t none) {
    if (bin == kNoVoxel) return none;
    const uint32_t x = bin & 31, w = bin >> 5;  // w: word index, (t * 8 + z) * 8 + y in its tile
    const uint32_t y = w & 7, z = (w >> 3) & 7, t = (w >> 6) & ((1u << logBT) - 1), tile = w >> (6 + logBT);
    const uint32_t sub = (y >> 2) | ((z >> 2) << 1) | ((x >> 3) << 2) | ((t >> 2) << 4);
    return (tile << (2 + logBT)) | sub;
}

// A wave holds 64 consecutive steps; consecutive steps of a trajectory mostly
// share a tile, so lanes split into runs of one key and only a run's first
// lane (head) touches the key's counter.
struct KeyRun {
    int head, len;
};

__device__ __forceinline__ KeyRun key_run(uint32_t key) {
    const int lane = threadIdx.x & 63;
    const uint32_t prev = (uint32_t)__shfl_up((int)key, 1);
    const unsigned long long starts = __ballot(lane == 0 || prev != key);
    const unsigned long long later = lane == 63 ? 0ull : starts >> (lane + 1);
    KeyRun r;
    r.len = later ? __builtin_ctzll(later) + 1 : 64 - lane;
    const unsigned long long upto = lane == 63 ? starts : starts & ((2ull << lane) - 1);
    r.head = 63 - __builtin_clzll(upto);  // lane 0 always starts a run
    return r;
}

__global__ __launch_bounds__(256) void k_order_count(const uint32_t* __restrict__ bins, uint64_t Qpad,
                                                     int Tpad, int T, int logBT, uint32_t none,
                                                     uint32_t* __restrict__ cnt) {
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    for (uint64_t w = (blockIdx.x * (uint64_t)blockDim.x + threadIdx.x) >> 6; w * 64 < Qpad; w += nwaves) {
        const uint64_t e = w * 64 + (threadIdx.x & 63);
        const bool step = e < Qpad && (int)(e % (uint64_t)Tpad) < T;
        const uint32_t key = step ? order_key(bins[e], logBT, none) : kSkip;
        const KeyRun r = key_run(key);
        if (key != kSkip && r.head == (int)(threadIdx.x & 63)) atomicAdd(&cnt[key], (uint32_t)r.len);
    }
}

// Exclusive prefix of the 256 values of a block; `total` gets their sum.
__device__ __forceinline__ uint32_t block_scan256(uint32_t v, uint32_t* s_w, uint32_t& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    uint32_t base = 0;
    for (int i = 0; i < wave; ++i) base += s_w[i];
    total = s_w[0] + s_w[1] + s_w[2] + s_w[3];
    __syncthreads();
    return base + x - v;
}

// Counts -> exclusive offsets, in place, over n buckets: per-block sums of
// consecutive ranges, one block scans them, each block writes its offsets.
__global__ __launch_bounds__(256) void k_order_sums(const uint32_t* __restrict__ cnt, uint32_t n,
                                                    uint32_t* __restrict__ bsum) {
    const uint32_t per = (n + kScanBlocks - 1) / kScanBlocks;
    const uint32_t i0 = blockIdx.x * per, i1 = min(n, i0 + per);
    uint32_t c = 0;
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += blockDim.x) c += cnt[i];
    for (int o = 32; o > 0; o >>= 1) c += (uint32_t)__shfl_xor((int)c, o);
    __shared__ uint32_t s_w[4];
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) bsum[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

__global__ __launch_bounds__(1024) void k_order_top(uint32_t* __restrict__ bsum) {
    __shared__ uint32_t s_w[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t v = bsum[threadIdx.x];
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) s_w[wave] = x;
    __syncthreads();
    uint32_t base = 0;
    for (int i = 0; i < wave; ++i) base += s_w[i];
    bsum[threadIdx.x] = base + x - v;
}

__global__ __launch_bounds__(256) void k_order_offsets(uint32_t* __restrict__ cnt, uint32_t n,
                                                       const uint32_t* __restrict__ bsum) {
    __shared__ uint32_t s_w[4];
    const uint32_t per = (n + kScanBlocks - 1) / kScanBlocks;
    const uint32_t i0 = blockIdx.x * per, i1 = min(n, i0 + per);
    uint32_t base = bsum[blockIdx.x];
    for (uint32_t b0 = i0; b0 < i1; b0 += blockDim.x) {  // block-uniform
        const uint32_t i = b0 + threadIdx.x;
        const uint32_t v = i < i1 ? cnt[i] : 0u;
        uint32_t total;
        const uint32_t ex = block_scan256(v, s_w, total);
        if (i < i1) cnt[i] = base + ex;
        base += total;
    }
}

// A block takes 64 particles x 64 steps.  First a wave walks a particle's steps
// (bins are [P][Tpad]: one line, and runs of one key share an atomic) and leaves
// their places in LDS; then a wave walks 64 particles at one step, so that the
// positions, values and places, all [T][P], are read and written in whole lines:
// 13.9 ms for 2.7e8 steps (with lanes along the steps each of them cost a line
// per lane: 20 to 24 ms).  The steps are a grid dimension too: 64 particles of 40,000
// steps 255 us, 11,900 with a block per 64 particles walking them all.
constexpr int kOrderP = 64, kOrderT = 64;
__global__ __launch_bounds__(256) void k_order_scatter(const uint32_t* __restrict__ bins, int Tpad, int T, int rate,
                                                       int logBT, uint32_t none, int64_t P, uint32_t* __restrict__ cur,
                                                       uint32_t* __restrict__ order, const float* __restrict__ xyz,
                                                       const float* __restrict__ attr, float4* __restrict__ spos,
                                                       float* __restrict__ sattr) {
    __shared__ uint32_t s_at[kOrderP][kOrderT + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t p0 = (int64_t)blockIdx.x * kOrderP;
    const int t0 = blockIdx.y * kOrderT;
    for (int j = wave; j < kOrderP && p0 + j < P; j += 4) {
        const int t = t0 + lane;
        const uint32_t key = t < T ? order_key(bins[(uint64_t)(p0 + j) * Tpad + t], logBT, none) : kSkip;
        const KeyRun r = key_run(key);
        uint32_t at = 0;
        if (key != kSkip && r.head == lane) at = atomicAdd(&cur[key], (uint32_t)r.len);
        s_at[j][lane] = (uint32_t)__shfl((int)at, r.head) + (uint32_t)(lane - r.head);
    }
    __syncthreads();
    const int64_t p = p0 + lane;
    for (int k = wave; k < kOrderT && t0 + k < T; k += 4) {
        if (p >= P) continue;
        const int t = t0 + k;
        const uint32_t at = s_at[lane][k];
        const uint64_t i = (uint64_t)t * P + p;
        order[i] = at;  // position of the step in the visiting order
        spos[at] = make_float4(xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2], __fdiv_rn((float)t, (float)rate));
        sattr[at] = attr[i];
    }
}

}  // namespace

// out[q] = in[pos[q]] over [T][P].  A block takes 64 particles x 64 steps: the
// places are read and the labels written with lanes along the particles (whole
// lines), the gather between them runs along each particle's steps, whose
// neighbours mostly lie side by side in the visiting order: 4.4 ms for 2.7e8
// labels, 5.2 ms gathered with lanes along the particles.
__global__ __launch_bounds__(256) void k_slic_unsort(const int32_t* __restrict__ in, const uint32_t* __restrict__ pos,
                                                     int T, int64_t P, int32_t* __restrict__ out) {
    __shared__ uint32_t s_v[kOrderP][kOrderT + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t p0 = (int64_t)blockIdx.x * kOrderP;
    const int t0 = blockIdx.y * kOrderT;
    const int64_t p = p0 + lane;
    for (int k = wave; k < kOrderT && t0 + k < T; k += 4)
        if (p < P) s_v[lane][k] = pos[(uint64_t)(t0 + k) * P + p];
    __syncthreads();
    for (int j = wave; j < kOrderP && p0 + j < P; j += 4)
        if (t0 + lane < T) s_v[j][lane] = (uint32_t)in[s_v[j][lane]];
    __syncthreads();
    for (int k = wave; k < kOrderT && t0 + k < T; k += 4)
        if (p < P) out[(uint64_t)(t0 + k) * P + p] = (int32_t)s_v[lane][k];
}

// Trajectory segments of the features (Section 3.4): a particle-step keeps
// its feature id when the same particle lies in that feature at t - 1 or
// t + 1 (so that runs of two or more consecutive steps are drawn), else -1.
// In place on point labels [T][P]: a thread owns one particle and reads its
// step t + 1 before it writes step t.  feat[centre] -> feature id.
__global__ __launch_bounds__(256) void k_slic_segments(int32_t* __restrict__ lab, const int32_t* __restrict__ feat,
                                                      int T, int64_t P) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < P; p += stride) {
        auto fid = [&](int t) -> int32_t {
            const int32_t l = lab[(int64_t)t * P + p];
            return l >= 0 ? feat[l] : -1;
        };
        int32_t prev = -1, cur = fid(0);
        for (int t = 0; t < T; ++t) {
            const int32_t next = t + 1 < T ? fid(t + 1) : -1;
            lab[(int64_t)t * P + p] = cur >= 0 && (cur == prev || cur == next) ? cur : -1;
            prev = cur;
            cur = next;
        }
    }
}

void launch_slic_segments(int32_t* lab, const int32_t* feat, int T, int64_t P, hipStream_t st) {
    if (T <= 0 || P <= 0) return;
    const unsigned g = (unsigned)std::min<int64_t>((P + 255) / 256, 16384);
    hipLaunchKernelGGL(k_slic_segments, dim3(g), dim3(256), 0, st, lab, feat, T, P);
}

void launch_slic_unsort(const int32_t* in, const uint32_t* order, int T, int64_t P, int32_t* out, hipStream_t st) {
    if (T <= 0 || P <= 0) return;
    hipLaunchKernelGGL(k_slic_unsort, dim3((unsigned)((P + kOrderP - 1) / kOrderP), (unsigned)((T + kOrderT - 1) / kOrderT)),
                       dim3(256), 0, st, in, order, T, P, out);
}

int launch_slic_order(const uint32_t* bins, const float* xyz, const float* attr, int64_t P, int Tpad,
                      int T, int r, int logBT, uint32_t ntiles, uint32_t* scratch, uint32_t* order, float4* spos,
                      float* sattr, hipStream_t st) {
    const uint64_t Qpad = (uint64_t)P * Tpad;
    const uint32_t none = slic_order_keys(ntiles, logBT) - 1;  // the last bucket: steps in no voxel
    const uint32_t nb = none + 1;
    uint32_t* cnt = scratch;
    uint32_t* bsum = scratch + nb + 1;
    launch_fill_u32(cnt, 0, nb, st);
    const unsigned g = (unsigned)std::min<uint64_t>((Qpad + 255) / 256, 8192);
    hipLaunchKernelGGL(k_order_count, dim3(g), dim3(256), 0, st, bins, Qpad, Tpad, T, logBT, none, cnt);
    hipLaunchKernelGGL(k_order_sums, dim3(kScanBlocks), dim3(256), 0, st, cnt, nb, bsum);
    hipLaunchKernelGGL(k_order_top, dim3(1), dim3(kScanBlocks), 0, st, bsum);
    hipLaunchKernelGGL(k_order_offsets, dim3(kScanBlocks), dim3(256), 0, st, cnt, nb, bsum);
    const dim3 chunks((unsigned)((P + kOrderP - 1) / kOrderP), (unsigned)((T + kOrderT - 1) / kOrderT));
    hipLaunchKernelGGL(k_order_scatter, chunks, dim3(256), 0, st, bins, Tpad, T,
                       r, logBT, none, P, cnt, order, xyz, attr, spos, sattr);
    return (int)hipGetLastError();
}

// Box shape of the field pass.  The wave box of 8 x 4 x 4 x 2 samples is compact
// in the distance (time counts c_f times) and reads whole 32-byte sectors; a
// planar grid gives z's share to y and t.  Four waves lie along x, so that a
// block reads whole 128-byte lines, unless the grid is too narrow for that.  A
// block takes four wave boxes per wave, which spreads its list over 4,096
// samples, as long as that leaves 2,048 blocks (8 per CU); below that one.
static FieldBox field_box(const DevS& s) {
    FieldBox b{};
    b.ly = s.Z > 1 ? 2 : 3;
    b.lz = s.Z > 1 ? 2 : 0;
    b.lt = s.Z > 1 ? 1 : 2;
    b.wx = s.X > 16 ? 2 : (s.X > 8 ? 1 : 0);
    b.vec = (s.X & 3) == 0;
    auto shape = [&](int iy, int iz, int it) {
        b.iy = iy;
        b.iz = iz;
        b.it = it;
        b.nx = (s.X + b.ex() - 1) / b.ex();
        b.ny = (s.Y + b.ey() - 1) / b.ey();
        b.nz = (s.Z + b.ez() - 1) / b.ez();
        b.nt = (s.T + b.et() - 1) / b.et();
        return (uint64_t)b.nx * b.ny * b.nz * b.nt;
    };
    const uint64_t big = s.Z > 1 ? shape(1, 1, 0) : shape(b.wx > 0, 0, 1);
    if (big < 2048) shape(0, 0, 0);
    return b;
}

// Points per thread of the point pass: four, while that leaves 2,048 blocks.
static int points_per_thread(const DevS& s) { return (uint64_t)s.Tp * s.P >= 2048ull * kBlock * kPer ? kPer : 1; }

uint32_t slic_boxes(const DevS& s) {
    const FieldBox b = field_box(s);
    return (uint32_t)b.nx * b.ny * b.nz * b.nt +
           blocks_for((uint64_t)s.Tp * s.P, (uint64_t)kBlock * points_per_thread(s));
}

template <int ASSIGN>
static void launch_pass(const DevS& s, hipStream_t st) {
    const uint64_t Q = (uint64_t)s.Tp * s.P;
    const FieldBox b = field_box(s);
    const uint32_t nf = (uint32_t)b.nx * b.ny * b.nz * b.nt;
    const int per = points_per_thread(s);
    const uint32_t np = blocks_for(Q, (uint64_t)kBlock * per);
    if (per == 1 && nf < 2048) {
        hipLaunchKernelGGL(k_slic_both<ASSIGN>, dim3(nf + np), dim3(kBlock), 0, st, s, b, nf);
    } else {
        hipLaunchKernelGGL(k_slic_field<ASSIGN>, dim3(nf), dim3(kBlock), 0, st, s, b);
        if (Q && per == 1) hipLaunchKernelGGL((k_slic_points<ASSIGN, 1>), dim3(np), dim3(kBlock), 0, st, s, nf);
        else if (Q) hipLaunchKernelGGL((k_slic_points<ASSIGN, kPer>), dim3(np), dim3(kBlock), 0, st, s, nf);
    }
    hipLaunchKernelGGL(k_slic_rest<ASSIGN>, dim3(std::min(nf + np, 2048u)), dim3(kBlock), 0, st, s, b, nf,
                       (uint32_t)(kBlock * per));
}

void launch_slic_begin(const DevS& s, hipStream_t st) {
    const unsigned g = (unsigned)std::min<uint64_t>(blocks_for((uint64_t)s.copies * s.K * kSlicAcc, 256), 2048);
    hipLaunchKernelGGL(k_slic_begin, dim3(g), dim3(256), 0, st, s);
    launch_pass<0>(s, st);
    hipLaunchKernelGGL(k_slic_update, dim3(blocks_for((uint64_t)s.K, 256)), dim3(256), 0, st, s, 1);
}

void launch_slic_iteration(const DevS& s, hipStream_t st) {
    launch_pass<1>(s, st);
    hipLaunchKernelGGL(k_slic_update, dim3(blocks_for((uint64_t)s.K, 256)), dim3(256), 0, st, s, 0);
}

int launch_slic_merge(const DevS& s, const DevM& m, hipStream_t st) {
    const dim3 gk(blocks_for((uint64_t)m.K, 256)), b256(256);
    const uint64_t Q = (uint64_t)s.Tp * s.P;
    hipLaunchKernelGGL(k_merge_init, gk, b256, 0, st, s, m);
    const int tile = m.K <= kMergeSmall ? 64 : 256;
    const unsigned nt = (unsigned)((m.K + tile - 1) / tile);
    if (tile == 64) hipLaunchKernelGGL(k_merge_pairs<64>, dim3(nt, nt), dim3(256), 0, st, s, m);
    else hipLaunchKernelGGL(k_merge_pairs<256>, dim3(nt, nt), dim3(256), 0, st, s, m);
    hipLaunchKernelGGL(k_merge_flatten, gk, b256, 0, st, s, m);
    hipLaunchKernelGGL(k_feature_sums, gk, b256, 0, st, s, m);
    hipLaunchKernelGGL(k_feature_means, gk, b256, 0, st, s, m);
    const FieldBox b = field_box(s);
    hipLaunchKernelGGL(k_feature_field, dim3((uint32_t)b.nx * b.ny * b.nz * b.nt), dim3(kBlock), 0, st, s, m, b);
    if (Q) hipLaunchKernelGGL(k_feature_points, dim3(blocks_for(Q, kBlock * kPer)), dim3(kBlock), 0, st, s, m);
    hipLaunchKernelGGL(k_feature_fold, gk, b256, 0, st, m);
    hipLaunchKernelGGL(k_feature_write, gk, b256, 0, st, m);
    return (int)hipGetLastError();
}

}  // namespace mf4d
