// Batched growing: up to 256 queries (each its own seeds and criteria) as the
// bit-planes of one 256-bit label per node, grown together in one pass over
// the data.  Query q lives in bit (q & 31) of word (q >> 5) of every node.
//
// Admissibility of a value v for all queries at once: with the lower bounds
// sorted ascending, {q : lo_q <= v} is the first rank_lo(v) queries of that
// order, a prefix mask read from a table; likewise for the upper bounds sorted
// descending.  The node's 256-bit mask is the AND of the two table rows.
//
// The two ranks of every voxel-step and particle-step (rank_lo | rank_hi <<
// 16) are computed once per grow, when its admissibility is first read, and
// kept: sweeps, pulls and closes rebuild a node's 256-bit mask from them with
// two rows of the prefix tables (staged in LDS), no search.  A particle-step
// that can exchange members with its voxel (some query admits both) is coupled:
// a bit beside its ranks says so, and the coupled steps are listed by tile.
//
// Field labels are grown in place in the caller's [V][8] output (canonical
// voxel order); particle labels in the caller's [T][P][8] output.  Work is
// organised in 4D tiles of 512 voxel-steps (a power-of-two extent per axis,
// chosen per context, e.g. 8 x 4 x 4 x 4).  A round sweeps the tiles of its
// work list, each handing what it gained to its own coupled steps; closes the
// trajectories of the particles that gained, pushing into their voxels; and
// lists the tiles flagged meanwhile (double-buffered by round parity).  A tile is flagged with the faces
// across which its neighbours gained members: its visit reads only those.
#include "mf4d_internal.h"
#include "batched.h"

namespace mf4d {

namespace {

constexpr int kWave = 64;
__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

struct Mask8 {
    uint32_t w[8];
};

// #{i : s[i] <= v} for s ascending (n <= 256); NaN v gives 0.
// The predicate holds on a prefix of s: its length by halving steps of
// fixed sizes (every lane takes the same steps: no divergence, one LDS read
// each).
__device__ __forceinline__ int rank_le(const float* s, int n, float v) {
    if (n <= 0) return 0;
    int pos = 0;
    for (int step = 1 << (31 - __clz(n)); step > 0; step >>= 1)
        if (pos + step <= n && s[pos + step - 1] <= v) pos += step;
    return pos;
}
// #{i : s[i] >= v} for s descending.
__device__ __forceinline__ int rank_ge(const float* s, int n, float v) {
    if (n <= 0) return 0;
    int pos = 0;
    for (int step = 1 << (31 - __clz(n)); step > 0; step >>= 1)
        if (pos + step <= n && s[pos + step - 1] >= v) pos += step;
    return pos;
}

// Tables: sorted bounds and prefix masks, for one sample type.
struct BandTables {
    const float* lo_sorted;  // ascending, Q
    const float* hi_sorted;  // descending, Q
    const uint32_t* lo_mask; // [Q+1][8]
    const uint32_t* hi_mask; // [Q+1][8]
};

__device__ __forceinline__ Mask8 band_mask(const BandTables& tb, int Q, float v) {
    const int rl = rank_le(tb.lo_sorted, Q, v);
    const int rh = rank_ge(tb.hi_sorted, Q, v);
    Mask8 m;
#pragma unroll
    for (int k = 0; k < 8; ++k) m.w[k] = tb.lo_mask[rl * 8 + k] & tb.hi_mask[rh * 8 + k];
    return m;
}

// Prefix-mask tables of one sample type staged in LDS: lo rows then hi rows,
// [257][8] words each, of which the Q + 1 rows in use are copied.
constexpr int kLdsTab = 2 * 257 * 8;

__device__ __forceinline__ void stage_tables(const DevB& d, int type, uint32_t* s_tab) {
    const uint4* src = reinterpret_cast<const uint4*>(d.tab + 1024) + (size_t)type * 2 * 257 * 2;
    uint4* dst = reinterpret_cast<uint4*>(s_tab);
    for (int i = threadIdx.x; i < (d.Q + 1) * 2; i += blockDim.x) {
        dst[i] = src[i];
        dst[257 * 2 + i] = src[257 * 2 + i];
    }
}

// Packed ranks: rank_lo in the low nine bits (at most 256), rank_hi from bit 16; bit
// 15 of a particle-step's: coupled.
constexpr uint32_t kRankLo = 0x1FFu, kCoupled = 1u << 15;
// Word k of the mask of a node with packed ranks r, from staged tables.
__device__ __forceinline__ uint32_t rank_word(const uint32_t* s_tab, uint32_t r, int k) {
    return s_tab[(r & kRankLo) * 8 + k] & s_tab[257 * 8 + (r >> 16) * 8 + k];
}

__device__ __forceinline__ BandTables field_tables(const DevB& d) {
    return BandTables{d.tab, d.tab + 256, reinterpret_cast<const uint32_t*>(d.tab + 1024),
                      reinterpret_cast<const uint32_t*>(d.tab + 1024) + 257 * 8};
}

__device__ __forceinline__ uint32_t btile_of(const DevB& d, int x, int y, int z, int t) {
    return ((uint32_t)((t >> d.lt) * d.NZb + (z >> d.lz)) * d.NYb + (y >> d.ly)) * d.NXb + (x >> d.lx);
}

__device__ __forceinline__ void btile_coords(const DevB& d, uint32_t tile, int& bx, int& by, int& bz,
                                             int& bt) {
    bx = tile % d.NXb;
    tile /= d.NXb;
    by = tile % d.NYb;
    tile /= d.NYb;
    bz = tile % d.NZb;
    bt = tile / d.NZb;
}

__device__ __forceinline__ uint64_t vindex(const DevB& d, int x, int y, int z, int t) {
    return (((uint64_t)t * d.Z + z) * d.Y + y) * d.X + x;
}

// Canonical voxel of a tile-layout bit position (the single-query binning).
__device__ __forceinline__ void bit_to_xyzt(const Geom& g, uint32_t b, int& x, int& y, int& z,
                                            int& t) {
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
    x = tx * 32 + (b & 31);
    y = ty * 8 + (wi & 7);
    z = tz * 8 + ((wi >> 3) & 7);
    t = (tt << g.logBT) + (wi >> 6);
}

// Scheduling flags a tile for the round of parity `par` (bit f: its neighbour
// across face f gained members there, faces in the order x-, x+, y-, .. t+;
// kOwn: it gained members itself outside a sweep) without a round trip to wait
// for; kb_compact turns the flags into that round's work list, dropping tiles
// without an admissible node.
constexpr uint32_t kOwn = 1u << 8;
__device__ __forceinline__ void bschedule(const DevB& d, uint32_t tile, int par, uint32_t bits) {
    atomicOr(&d.dirty[par * d.NTB + tile], bits);
}

// A voxel that gained members outside a sweep: its tile and the tiles whose face
// it touches.
__device__ __forceinline__ void bmark_voxel(const DevB& d, int x, int y, int z, int t, int par) {
    const uint32_t tile = btile_of(d, x, y, z, t);
    bschedule(d, tile, par, kOwn);
    const uint32_t sy = d.NXb, sz = d.NXb * d.NYb, st = sz * d.NZb;
    const int mx = (1 << d.lx) - 1, my = (1 << d.ly) - 1, mz = (1 << d.lz) - 1, mt = (1 << d.lt) - 1;
    if ((x & mx) == 0 && x > 0) bschedule(d, tile - 1, par, 1u << 1);
    if ((x & mx) == mx && x + 1 < d.X) bschedule(d, tile + 1, par, 1u << 0);
    if ((y & my) == 0 && y > 0) bschedule(d, tile - sy, par, 1u << 3);
    if ((y & my) == my && y + 1 < d.Y) bschedule(d, tile + sy, par, 1u << 2);
    if ((z & mz) == 0 && z > 0) bschedule(d, tile - sz, par, 1u << 5);
    if ((z & mz) == mz && z + 1 < d.Z) bschedule(d, tile + sz, par, 1u << 4);
    if ((t & mt) == 0 && t > 0) bschedule(d, tile - st, par, 1u << 7);
    if ((t & mt) == mt && t + 1 < d.T) bschedule(d, tile + st, par, 1u << 6);
}

// Coordinates of a canonical voxel index.
__device__ __forceinline__ void voxel_coords(const DevB& d, uint32_t v, int& x, int& y, int& z, int& t) {
    x = (int)(v % (uint32_t)d.X);
    v /= (uint32_t)d.X;
    y = (int)(v % (uint32_t)d.Y);
    v /= (uint32_t)d.Y;
    z = (int)(v % (uint32_t)d.Z);
    t = (int)(v / (uint32_t)d.Z);
}

// Lane i of eight (a tile's faces in order) flags the neighbour across face i
// of a tile whose nodes there gained members (faces: those faces).
__device__ __forceinline__ void bschedule_face(const DevB& d, uint32_t tile, int bx, int by, int bz, int bt, int i,
                                               uint32_t faces, int par) {
    if (!((faces >> i) & 1u)) return;
    const uint32_t sy = d.NXb, sz = d.NXb * d.NYb, st = sz * d.NZb;
    const int axis = i >> 1;
    const int b = axis == 0 ? bx : axis == 1 ? by : axis == 2 ? bz : bt;
    const int n = axis == 0 ? d.NXb : axis == 1 ? d.NYb : axis == 2 ? d.NZb : d.NTb;
    const uint32_t st_a = axis == 0 ? 1u : axis == 1 ? sy : axis == 2 ? sz : st;
    if ((i & 1) ? b + 1 < n : b > 0) bschedule(d, (i & 1) ? tile + st_a : tile - st_a, par, 1u << (i ^ 1));
}

// ---------------------------------------------------------------------------

// The sorted bounds of one sample type staged in LDS (lo ascending, then hi
// descending, 256 each), for the rank searches of a whole block.
__device__ __forceinline__ void stage_bounds(const DevB& d, int type, float* s_b) {
    for (int i = threadIdx.x; i < 512; i += blockDim.x) s_b[i] = d.tab[512 * type + i];
}

// Clear the field planes, record every voxel-step's ranks, mark tiles that hold
// a node admissible for some query.  A block takes 1,024 voxel-steps at a time,
// four a thread, whose rank searches interleave, and stores their 32 KB of planes
// in order, 16 bytes a lane.  Bound by those stores.
// 128^3 x 32: 612 us; 760 with a thread storing its own nodes' 32 bytes.
__global__ __launch_bounds__(256) void kb_admit_field(DevB d) {
    __shared__ float s_b[512];
    stage_bounds(d, 0, s_b);
    __syncthreads();
    const uint32_t* ftab = reinterpret_cast<const uint32_t*>(d.tab + 1024);
    const uint64_t V = (uint64_t)d.X * d.Y * d.Z * d.T;
    constexpr int kU = 4, kStep = kU * 256;
    for (uint64_t b0 = (uint64_t)blockIdx.x * kStep; b0 < V; b0 += (uint64_t)gridDim.x * kStep) {
        float f[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t v = b0 + u * 256 + threadIdx.x;
            f[u] = v < V ? __builtin_nontemporal_load(d.field + v) : 0.0f;
        }
        const uint64_t n4 = (V - b0 < (uint64_t)kStep ? V - b0 : (uint64_t)kStep) * 2;  // 16-byte pieces
        uint4* o = reinterpret_cast<uint4*>(d.fplanes + b0 * 8);
#pragma unroll
        for (int u = 0; u < 2 * kU; ++u) {
            const uint32_t i = u * 256 + threadIdx.x;
            if (i < n4) o[i] = make_uint4(0, 0, 0, 0);
        }
        uint32_t r[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u)
            r[u] = (uint32_t)rank_le(s_b, d.Q, f[u]) | ((uint32_t)rank_ge(s_b + 256, d.Q, f[u]) << 16);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t v = b0 + u * 256 + threadIdx.x;
            if (v >= V) continue;
            d.vrank[v] = r[u];
            uint32_t any = 0;
            if ((r[u] & 0xFFFFu) && (r[u] >> 16)) {
#pragma unroll
                for (int k = 0; k < 8; ++k) any |= rank_word(ftab, r[u], k);
            }
            if (any) {
                int x, y, z, t;
                voxel_coords(d, (uint32_t)v, x, y, z, t);
                d.active[btile_of(d, x, y, z, t)] = 1;
            }
        }
    }
}

// Clear the particle planes, record every particle-step's ranks and whether it is
// coupled (it lies in a voxel and some query admits both), counted for the voxel's
// tile.  Four steps a thread, whose loads and searches interleave.
// 262,144 x 32: 98 us, and 22 to list the coupled steps; 229 with a list appended
// to by whole blocks.
__global__ __launch_bounds__(256) void kb_admit_particles(DevB d) {
    __shared__ float s_b[512];
    stage_bounds(d, 1, s_b);
    __syncthreads();
    const uint32_t* ftab = reinterpret_cast<const uint32_t*>(d.tab + 1024);
    const uint32_t* ptab = ftab + 2 * 257 * 8;
    const uint64_t n = (uint64_t)d.P * d.Tpad;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t np = (uint64_t)d.Tp * d.P * 2;  // uint4 per particle-step: 2
    const uint64_t tid = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    for (uint64_t i = tid; i < np; i += stride) reinterpret_cast<uint4*>(d.pplanes)[i] = make_uint4(0, 0, 0, 0);
    constexpr int kU = 4;
    for (uint64_t e0 = tid; e0 < n; e0 += kU * stride) {
        float a[kU];
        uint32_t b[kU], r[kU], vr[kU], vox[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t e = e0 + u * stride;
            a[u] = 0.0f;
            b[u] = kNoVoxel;
            if (e < n) {
                a[u] = d.attr_t[e];
                b[u] = d.bins[e];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            r[u] = (uint32_t)rank_le(s_b, d.Q, a[u]) | ((uint32_t)rank_ge(s_b + 256, d.Q, a[u]) << 16);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            vox[u] = kNoVoxel;
            vr[u] = 0;
            if (b[u] != kNoVoxel && (r[u] & 0xFFFFu) && (r[u] >> 16)) {
                int x, y, z, t;
                bit_to_xyzt(d.g, b[u], x, y, z, t);
                vox[u] = (uint32_t)vindex(d, x, y, z, t);
                vr[u] = d.vrank[vox[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t e = e0 + u * stride;
            if (e >= n) continue;
            uint32_t any = 0;
            if ((vr[u] & 0xFFFFu) && (vr[u] >> 16)) {
#pragma unroll
                for (int k = 0; k < 8; ++k) any |= rank_word(ptab, r[u], k) & rank_word(ftab, vr[u], k);
            }
            if (any) {
                int x, y, z, t;
                voxel_coords(d, vox[u], x, y, z, t);
                atomicAdd(&d.tcnt[btile_of(d, x, y, z, t)], 1u);
            }
            d.prank[e] = r[u] | (any ? kCoupled : 0u);
        }
    }
}

// The coupled steps into their tiles' ranges of the list (kb_compact has given
// every tile the end of its range, which becomes its start here).
__global__ __launch_bounds__(256) void kb_couple(DevB d) {
    const uint32_t n = (uint32_t)((uint64_t)d.P * d.Tpad);
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        const uint32_t b = d.bins[e];
        if (!(d.prank[e] & kCoupled)) continue;
        int x, y, z, t;
        bit_to_xyzt(d.g, b, x, y, z, t);
        d.clist[atomicSub(&d.tbase[btile_of(d, x, y, z, t)], 1u) - 1] = make_uint2(e, (uint32_t)vindex(d, x, y, z, t));
    }
}

__global__ void kb_seeds(DevB d, const int32_t* __restrict__ seeds, int64_t S) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= S) return;
    const int32_t* s = seeds + 5 * i;
    const int x = s[0], y = s[1], z = s[2], t = s[3], q = s[4];
    const uint64_t v = vindex(d, x, y, z, t);
    const Mask8 m = band_mask(field_tables(d), d.Q, d.field[v]);
    const uint32_t bit = 1u << (q & 31);
    if (m.w[q >> 5] & bit) {
        if (!(atomicOr(&d.fplanes[v * 8 + (q >> 5)], bit) & bit)) bmark_voxel(d, x, y, z, t, 0);
    } else {
        atomicAdd(&d.counters[BC_DROPPED], 1u);
    }
}

// Lane moves (DPP), register only: the neighbour in a group of four lanes (its
// first and last lane receive their own value), and four
// lanes up or down in a row of 16 (0 from outside the row).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_ones(uint32_t v) {  // all ones from outside the row
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, 0xF, 0xF, false);
}
constexpr int kQuadPrev = 0x90, kQuadNext = 0xF9, kRowPrev4 = 0x114, kRowNext4 = 0x104;

// A list kept as kBSubs sub-lists seen as one: the sub-lists' prefix sums.
__device__ __forceinline__ void stage_list(const uint32_t* cnt, uint32_t* s_pref) {
    if (threadIdx.x < kBSubs) {
        // the first wave scans the sub-list lengths
        const uint32_t c = cnt[threadIdx.x * kBCntStride];
        uint32_t x = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if ((int)threadIdx.x >= o) x += y;
        }
        s_pref[threadIdx.x + 1] = x;
        if (threadIdx.x == 0) s_pref[0] = 0;
    }
    __syncthreads();
}
// The sub-list holding item w: the last j with s_pref[j] <= w.
__device__ __forceinline__ int sub_list(const uint32_t* s_pref, uint32_t w) {
    int lo = 0;
#pragma unroll
    for (int h = kBSubs / 2; h > 0; h >>= 1)
        if (s_pref[lo + h] <= w) lo += h;
    return lo;
}
__device__ __forceinline__ const uint32_t* work_counts(const DevB& d, int par) {
    return d.wcnt + (size_t)par * kBSubs * kBCntStride;
}
__device__ __forceinline__ uint2 work_item(const DevB& d, int par, const uint32_t* s_pref, uint32_t w) {
    const int j = sub_list(s_pref, w);
    return d.work[((size_t)par * kBSubs + j) * d.WCAPB + (w - s_pref[j])];
}
// A round's counters: rounds are queued ahead of the host, and a round whose
// work list is empty does nothing (recorded for its close).
__device__ __forceinline__ void begin_round(const DevB& d, uint32_t nwork) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        d.counters[BC_RACT] = nwork ? 1u : 0u;
        if (nwork) {
            d.counters[BC_ROUNDS] += 1u;
            d.stat64[S_TILE_VISITS] += nwork;
        }
    }
}

// A particle that gained, for the close: listed once.
__device__ __forceinline__ void list_particle(const DevB& d, uint32_t p) {
    const uint32_t pb = 1u << (p & 31);
    if (!(atomicOr(&d.pdirty[p >> 5], pb) & pb)) {
        const uint32_t j = p / d.DCAPB;
        d.dlist[j * d.DCAPB + atomicAdd(&d.dcnt[j * kBCntStride], 1u)] = p;
    }
}

// Word `word` of a swept tile handed to its coupled steps by 64 lanes (li: which):
// a step gains the queries for which its voxel is a member and it is admissible.
// Nothing else writes the word of these steps meanwhile.
__device__ __forceinline__ void pull_word(const DevB& d, uint32_t tile, uint32_t word, int li,
                                          const uint32_t* s_ptab) {
    const uint32_t n = d.tcnt[tile], base = d.tbase[tile];
    constexpr uint32_t kU = 4, W = 64;
    for (uint32_t i0 = li; i0 < n; i0 += kU * W) {
        uint2 ent[kU];
        uint32_t p[kU], m[kU], r[kU], lp[kU];
        uint64_t at[kU];
#pragma unroll
        for (uint32_t u = 0; u < kU; ++u) {
            const uint32_t i = i0 + u * W;
            ent[u] = d.clist[base + (i < n ? i : i0)];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            p[u] = ent[u].x / (uint32_t)d.Tpad;
            at[u] = ((uint64_t)(ent[u].x - p[u] * (uint32_t)d.Tpad) * d.P + p[u]) * 8 + word;
            m[u] = d.fplanes[(uint64_t)ent[u].y * 8 + word];
            r[u] = d.prank[ent[u].x];
            lp[u] = d.pplanes[at[u]];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t nw = m[u] & ~lp[u] & rank_word(s_ptab, r[u], word);
            if (nw && i0 + u * W < n) {
                d.pplanes[at[u]] = lp[u] | nw;
                list_particle(d, p[u]);
            }
        }
    }
}

// Four words of a swept tile handed to its coupled steps by a wave: as pull_word,
// with 16-byte reads and writes.
__device__ __forceinline__ uint4 rank_words4(const uint32_t* s_tab, uint32_t r, uint32_t k) {
    const uint4 a = *reinterpret_cast<const uint4*>(s_tab + (r & kRankLo) * 8 + k);
    const uint4 b = *reinterpret_cast<const uint4*>(s_tab + 257 * 8 + (r >> 16) * 8 + k);
    return make_uint4(a.x & b.x, a.y & b.y, a.z & b.z, a.w & b.w);
}
__device__ __forceinline__ void pull_words4(const DevB& d, uint32_t tile, uint32_t word, const uint32_t* s_ptab) {
    const uint32_t n = d.tcnt[tile], base = d.tbase[tile];
    for (uint32_t i = lane_id(); i < n; i += 64) {
        const uint2 ent = d.clist[base + i];
        const uint32_t p = ent.x / (uint32_t)d.Tpad;
        uint4* pp = reinterpret_cast<uint4*>(
            d.pplanes + ((uint64_t)(ent.x - p * (uint32_t)d.Tpad) * d.P + p) * 8 + word);
        const uint4 m = *reinterpret_cast<const uint4*>(d.fplanes + (uint64_t)ent.y * 8 + word);
        const uint4 a = rank_words4(s_ptab, d.prank[ent.x], word);
        const uint4 l = *pp;
        const uint4 g = make_uint4(l.x | (m.x & a.x), l.y | (m.y & a.y), l.z | (m.z & a.z), l.w | (m.w & a.w));
        if ((g.x ^ l.x) | (g.y ^ l.y) | (g.z ^ l.z) | (g.w ^ l.w)) {
            *pp = g;
            list_particle(d, p);
        }
    }
}

// Sweep of tiles with at least four nodes along x and along y.  A wave takes four
// words (128 queries) of one tile, a lane an x by y piece of one quarter of the
// tile along t (along z at an extent below four): eight nodes, in registers.  A
// line of nodes within a lane is closed by one pass up and one down; between lanes
// the words move by DPP, between quarters by lane permutes.  No barrier: a word's
// loop ends when it gained nothing in the wave (labels only grow).  Only nodes that
// admit a query of the words are read, and only the faces the tile is flagged for;
// what a tile gained it hands to its coupled steps.
// Bound by the chain list - ranks - labels and faces, and where many tiles wait by
// the vector memory unit, which takes a cycle for every lane's 32-byte sector
// whatever its width: a lane moves 16 bytes.  128^3 x 32, 256 queries, 67,600
// visits of 4 x 4 x 4 x 8 tiles: 1,330 us with the coupled steps; 1,770 with one
// word to 32 lanes (which is slower for 8 to 128 queries too: 64^3 x 16, 24
// queries, a whole call 567 us, here 451); 3,058, and 494 for the steps, with a
// block of 512 threads per tile passing eight words through LDS and reading every
// face.
template <int LX, int LY, int LZ, int LT>
__global__ __launch_bounds__(256) void kb_sweep_tiles(DevB d, int par) {
    constexpr bool kT = LT >= 2;  // the quarters lie along t
    constexpr int NX = 1 << (LX - 2), NY = 1 << (LY - 2), NZ = kT ? 1 << LZ : 1 << (LZ - 2),
                  NT = kT ? 1 << (LT - 2) : 1 << LT, N = 8;
    static_assert(LX >= 2 && LY >= 2 && (kT || LZ >= 2) && NX * NY * NZ * NT == N, "8 nodes a lane");
    // (a quarter's end lanes receive their own first or last layer: a neighbour, or the node itself)
    static_assert((kT ? NT : NZ) <= 2, "layers of a quarter");
    __shared__ __attribute__((aligned(16))) uint32_t s_ftab[kLdsTab];
    __shared__ __attribute__((aligned(16))) uint32_t s_ptab[kLdsTab];
    __shared__ uint32_t s_pref[kBSubs + 1];
    stage_list(work_counts(d, par), s_pref);
    const uint32_t nwork = s_pref[kBSubs];
    begin_round(d, nwork);
    const uint32_t ng = ((uint32_t)d.Q + 127) >> 7;
    const uint32_t items = nwork * ng;  // at most 2 x NTB
    if (blockIdx.x * 4 >= items) return;  // block-uniform
    stage_tables(d, 0, s_ftab);
    if (d.P > 0) stage_tables(d, 1, s_ptab);
    __syncthreads();
    const int lane = lane_id(), xl = lane & 3, yl = (lane >> 2) & 3, qr = lane >> 4;
    const int prev = qr > 0 ? lane - 16 : lane, next = qr < 3 ? lane + 16 : lane;
    const uint64_t sy = (uint64_t)d.X, sz = sy * d.Y, st = sz * d.Z;
    const uint4* zero = reinterpret_cast<const uint4*>(d.tab + 1024);  // row 0 of a mask table
    const uint32_t first = NX <= 2 || xl != 0 ? ~0u : 0u, last = NX <= 2 || xl != 3 ? ~0u : 0u;
    for (uint32_t it0 = blockIdx.x * 4 + (threadIdx.x >> 6); it0 < items; it0 += gridDim.x * 4) {
        const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)it0);
        const uint32_t w = ng == 2 ? it >> 1 : it, word = ng == 2 ? (it & 1) * 4 : 0;
        const uint2 e = work_item(d, par, s_pref, w);
        const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.x);
        const uint32_t flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.y);
        int bx, by, bz, bt;
        btile_coords(d, tile, bx, by, bz, bt);
        const int x0 = (bx << LX) + xl * NX, y0 = (by << LY) + yl * NY, z0 = (bz << LZ) + (kT ? 0 : qr * NZ),
                  t0 = (bt << LT) + (kT ? qr * NT : 0);
        const uint64_t v0 = vindex(d, x0, y0, z0, t0);
        auto off = [&](int j) {
            return (uint64_t)(j % NX) + (uint64_t)(j / NX % NY) * sy + (uint64_t)(j / (NX * NY) % NZ) * sz +
                   (uint64_t)(j / (NX * NY * NZ)) * st;
        };
        uint32_t rv[N], a[N][4], l[N][4], cnt[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const bool in = x0 + j % NX < d.X && y0 + j / NX % NY < d.Y && z0 + j / (NX * NY) % NZ < d.Z &&
                            t0 + j / (NX * NY * NZ) < d.T;
            rv[j] = 0;
            if (in) rv[j] = d.vrank[v0 + off(j)];
        }
        uint32_t adm = 0;  // bit j: node j admits one of the words' queries
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint4 m = rank_words4(s_ftab, rv[j], word);
            a[j][0] = m.x; a[j][1] = m.y; a[j][2] = m.z; a[j][3] = m.w;
            if (m.x | m.y | m.z | m.w) adm |= 1u << j;
        }
        uint4* fp = reinterpret_cast<uint4*>(d.fplanes + v0 * 8 + word);
        // node j's neighbour o nodes away (0 where the lane has none)
        auto read = [&](int j, bool has, int64_t o) {
            return *(has && ((adm >> j) & 1u) ? fp + ((int64_t)off(j) + o) * 2 : zero);
        };
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint4 v = read(j, true, 0);
            l[j][0] = v.x; l[j][1] = v.y; l[j][2] = v.z; l[j][3] = v.w;
            cnt[j] = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
        }
#define MF4D_FACE(FLAGS, COND, HAS, OFF)                                           \
    if (flags & (FLAGS)) {                                                         \
        uint4 h[N];                                                                \
        _Pragma("unroll") for (int j = 0; j < N; ++j) {                            \
            const int jx = j % NX, jy = j / NX % NY, jz = j / (NX * NY) % NZ, jt = j / (NX * NY * NZ); \
            (void)jx; (void)jy; (void)jz; (void)jt;                                \
            if (COND) h[j] = read(j, HAS, OFF);                                    \
            else h[j] = make_uint4(0, 0, 0, 0);                                    \
        }                                                                          \
        _Pragma("unroll") for (int j = 0; j < N; ++j) {                            \
            l[j][0] |= h[j].x & a[j][0];                                           \
            l[j][1] |= h[j].y & a[j][1];                                           \
            l[j][2] |= h[j].z & a[j][2];                                           \
            l[j][3] |= h[j].w & a[j][3];                                           \
        }                                                                          \
    }
        const bool xm = (flags & 1u) && xl == 0, xp = (flags & 2u) && xl == 3;
        const bool ym = (flags & 4u) && yl == 0, yp = (flags & 8u) && yl == 3;
        const bool qm = qr == 0, qp = qr == 3;
        if constexpr (NX == 1) {
            MF4D_FACE(3u, true, xm || xp, xm ? -1ll : 1ll)
        } else {
            MF4D_FACE(1u, jx == 0, xm, -1ll)
            MF4D_FACE(2u, jx == NX - 1, xp, 1ll)
        }
        if constexpr (NY == 1) {
            MF4D_FACE(12u, true, ym || yp, ym ? -(int64_t)sy : (int64_t)sy)
        } else {
            MF4D_FACE(4u, jy == 0, ym, -(int64_t)sy)
            MF4D_FACE(8u, jy == NY - 1, yp, (int64_t)sy)
        }
        MF4D_FACE(16u, jz == 0, kT || qm, -(int64_t)sz)
        MF4D_FACE(32u, jz == NZ - 1, kT || qp, (int64_t)sz)
        MF4D_FACE(64u, jt == 0, !kT || qm, -(int64_t)st)
        MF4D_FACE(128u, jt == NT - 1, !kT || qp, (int64_t)st)
#undef MF4D_FACE
        auto at = [](int jx, int jy, int jz, int jt) { return ((jt * NZ + jz) * NY + jy) * NX + jx; };
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t room = 0, src = 0, c = 0;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                room |= a[j][k] & ~l[j][k];
                src |= l[j][k];
                c += __popc(l[j][k]);
            }
            if (!__ballot(room) || !__ballot(src)) continue;  // nothing to gain, or nowhere to gain it from
            while (true) {
                // lines along t, z within the lane
#pragma unroll
                for (int r = 0; r < N / NT; ++r) {
#pragma unroll
                    for (int i = 1; i < NT; ++i) l[i * (N / NT) + r][k] |= l[(i - 1) * (N / NT) + r][k] & a[i * (N / NT) + r][k];
#pragma unroll
                    for (int i = NT - 2; i >= 0; --i)
                        l[i * (N / NT) + r][k] |= l[(i + 1) * (N / NT) + r][k] & a[i * (N / NT) + r][k];
                }
#pragma unroll
                for (int jt = 0; jt < NT; ++jt)
#pragma unroll
                    for (int r = 0; r < NX * NY; ++r) {
                        const int b = jt * NZ * NY * NX + r, s = NX * NY;
#pragma unroll
                        for (int i = 1; i < NZ; ++i) l[b + i * s][k] |= l[b + (i - 1) * s][k] & a[b + i * s][k];
#pragma unroll
                        for (int i = NZ - 2; i >= 0; --i) l[b + i * s][k] |= l[b + (i + 1) * s][k] & a[b + i * s][k];
                    }
#pragma unroll
                for (int jt = 0; jt < NT; ++jt)
#pragma unroll
                    for (int jz = 0; jz < NZ; ++jz) {
                        if constexpr (NX == 1 && NY == 1) {
                            const int j = at(0, 0, jz, jt);
                            uint32_t n = dpp<kQuadPrev>(l[j][k]);
                            n |= dpp<kQuadNext>(l[j][k]);
                            n |= dpp<kRowPrev4>(l[j][k]);
                            n |= dpp<kRowNext4>(l[j][k]);
                            l[j][k] |= n & a[j][k];
                        } else {
#pragma unroll
                            for (int jy = 0; jy < NY; ++jy) {
                                const int b = at(0, jy, jz, jt);
                                l[b][k] |= dpp<kQuadPrev>(l[b + NX - 1][k]) & a[b][k] & first;
#pragma unroll
                                for (int i = 1; i < NX; ++i) l[b + i][k] |= l[b + i - 1][k] & a[b + i][k];
                                l[b + NX - 1][k] |= dpp<kQuadNext>(l[b][k]) & a[b + NX - 1][k] & last;
#pragma unroll
                                for (int i = NX - 2; i >= 0; --i) l[b + i][k] |= l[b + i + 1][k] & a[b + i][k];
                            }
#pragma unroll
                            for (int jx = 0; jx < NX; ++jx) {
                                const int b = at(jx, 0, jz, jt), z = b + (NY - 1) * NX;
                                l[b][k] |= dpp<kRowPrev4>(l[z][k]) & a[b][k];
#pragma unroll
                                for (int i = 1; i < NY; ++i) l[b + i * NX][k] |= l[b + (i - 1) * NX][k] & a[b + i * NX][k];
                                l[z][k] |= dpp<kRowNext4>(l[b][k]) & a[z][k];
#pragma unroll
                                for (int i = NY - 2; i >= 0; --i)
                                    l[b + i * NX][k] |= l[b + (i + 1) * NX][k] & a[b + i * NX][k];
                            }
                        }
                    }
                // the layers where quarters meet
                constexpr int L = kT ? NX * NY * NZ : NX * NY;  // nodes between two layers
                uint32_t up[N], dn[N];
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const int i = kT ? j / (NX * NY * NZ) : j / (NX * NY) % NZ;  // layer of the quarter
                    if (i != 0) continue;
                    up[j] = (uint32_t)__shfl((int)l[j + ((kT ? NT : NZ) - 1) * L][k], prev);
                    dn[j] = (uint32_t)__shfl((int)l[j][k], next);
                }
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    const int i = kT ? j / (NX * NY * NZ) : j / (NX * NY) % NZ;
                    if (i != 0) continue;
                    const int z = j + ((kT ? NT : NZ) - 1) * L;
                    l[j][k] |= up[j] & a[j][k];
                    l[z][k] |= dn[j] & a[z][k];
                }
                uint32_t now = 0;
#pragma unroll
                for (int j = 0; j < N; ++j) now += __popc(l[j][k]);
                const bool grew = now != c;
                c = now;
                if (!__ballot(grew)) break;
            }
        }
        // The other words of these nodes are another wave's, and nothing else
        // writes them meanwhile: plain stores.
        uint32_t g = 0;  // bit j: node j gained
#pragma unroll
        for (int j = 0; j < N; ++j)
            if ((uint32_t)(__popc(l[j][0]) + __popc(l[j][1]) + __popc(l[j][2]) + __popc(l[j][3])) != cnt[j]) {
                fp[off(j) * 2] = make_uint4(l[j][0], l[j][1], l[j][2], l[j][3]);
                g |= 1u << j;
            }
        uint32_t f = 0;
        if (__ballot(g)) {
            uint32_t mx0 = 0, mx1 = 0, my0 = 0, my1 = 0, mz0 = 0, mz1 = 0, mt0 = 0, mt1 = 0;  // nodes on a face
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const int jx = j % NX, jy = j / NX % NY, jz = j / (NX * NY) % NZ, jt = j / (NX * NY * NZ);
                if (jx == 0) mx0 |= 1u << j;
                if (jx == NX - 1) mx1 |= 1u << j;
                if (jy == 0) my0 |= 1u << j;
                if (jy == NY - 1) my1 |= 1u << j;
                if (jz == 0) mz0 |= 1u << j;
                if (jz == NZ - 1) mz1 |= 1u << j;
                if (jt == 0) mt0 |= 1u << j;
                if (jt == NT - 1) mt1 |= 1u << j;
            }
            f = kOwn | (__ballot(xl == 0 && (g & mx0)) ? 1u : 0u) | (__ballot(xl == 3 && (g & mx1)) ? 2u : 0u) |
                (__ballot(yl == 0 && (g & my0)) ? 4u : 0u) | (__ballot(yl == 3 && (g & my1)) ? 8u : 0u) |
                (__ballot((kT || qm) && (g & mz0)) ? 16u : 0u) | (__ballot((kT || qp) && (g & mz1)) ? 32u : 0u) |
                (__ballot((!kT || qm) && (g & mt0)) ? 64u : 0u) | (__ballot((!kT || qp) && (g & mt1)) ? 128u : 0u);
            if (lane < 8) bschedule_face(d, tile, bx, by, bz, bt, lane, f, par ^ 1);
            // the nodes are read again by other lanes
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        }
        if (d.P > 0 && ((f | flags) & kOwn)) pull_words4(d, tile, word, s_ptab);
    }
}

// Sweep one tile (block of 512 threads, one voxel-step each) to a local fixed
// point: Jacobi steps through LDS over the 8 in-tile neighbours, the out-of-
// tile neighbours entering as fixed halos.  For tiles too thin for the sweep above.
__device__ void bsweep_tile(const DevB& d, uint2 item, int par, uint32_t* s_lab, uint32_t* s_flags,
                            const uint32_t* s_ftab, const uint32_t* s_ptab) {
    const uint32_t tile = item.x;
    int bx, by, bz, bt;
    btile_coords(d, tile, bx, by, bz, bt);
    const int tid = threadIdx.x;
    const int mx = (1 << d.lx) - 1, my = (1 << d.ly) - 1, mz = (1 << d.lz) - 1, mt = (1 << d.lt) - 1;
    const int sxl = 1, syl = 1 << d.lx, szl = 1 << (d.lx + d.ly), stl = 1 << (d.lx + d.ly + d.lz);
    const int xl = tid & mx, yl = (tid >> d.lx) & my, zl = (tid >> (d.lx + d.ly)) & mz,
              tl = tid >> (d.lx + d.ly + d.lz);
    const int x = (bx << d.lx) + xl, y = (by << d.ly) + yl, z = (bz << d.lz) + zl, t = (bt << d.lt) + tl;
    const bool in = x < d.X && y < d.Y && z < d.Z && t < d.T;
    if (tid == 0) {
        s_flags[0] = 0;
        s_flags[1] = 0;
        s_flags[2] = 0;
    }
    uint32_t a[8], l[8], h[8];  // a: the admissible queries per word
    const uint64_t v = in ? vindex(d, x, y, z, t) : 0;
    if (in) {
        const uint32_t rv = d.vrank[v];
        const uint4* lp = reinterpret_cast<const uint4*>(d.fplanes + v * 8);
        const uint4 l01 = lp[0], l23 = lp[1];
        l[0] = l01.x; l[1] = l01.y; l[2] = l01.z; l[3] = l01.w;
        l[4] = l23.x; l[5] = l23.y; l[6] = l23.z; l[7] = l23.w;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            a[k] = rank_word(s_ftab, rv, k);
            h[k] = 0;
        }
        // halos: neighbours outside the tile (inside the grid), each load
        // issued on its own condition (no indexed list: it would live in
        // scratch memory)
        const uint64_t sx = 1, sy = d.X, sz = (uint64_t)d.X * d.Y, st = sz * d.Z;
        auto halo = [&](bool has, uint64_t nv) {
            if (!has) return;
            const uint4* hp = reinterpret_cast<const uint4*>(d.fplanes + nv * 8);
            const uint4 h01 = hp[0], h23 = hp[1];
            h[0] |= h01.x; h[1] |= h01.y; h[2] |= h01.z; h[3] |= h01.w;
            h[4] |= h23.x; h[5] |= h23.y; h[6] |= h23.z; h[7] |= h23.w;
        };
        halo(xl == 0 && x > 0, v - sx);
        halo(xl == mx && x + 1 < d.X, v + sx);
        halo(yl == 0 && y > 0, v - sy);
        halo(yl == my && y + 1 < d.Y, v + sy);
        halo(zl == 0 && z > 0, v - sz);
        halo(zl == mz && z + 1 < d.Z, v + sz);
        halo(tl == 0 && t > 0, v - st);
        halo(tl == mt && t + 1 < d.T, v + st);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] = l[k] = h[k] = 0;
    }
    uint32_t grown = 0;  // some word of this node gained bits in this visit
    // in-tile neighbour thread ids (or -1)
    const int nx0 = xl > 0 ? tid - sxl : -1, nx1 = xl < mx ? tid + sxl : -1;
    const int ny0 = yl > 0 ? tid - syl : -1, ny1 = yl < my ? tid + syl : -1;
    const int nz0 = zl > 0 ? tid - szl : -1, nz1 = zl < mz ? tid + szl : -1;
    const int nt0 = tl > 0 ? tid - stl : -1, nt1 = tl < mt ? tid + stl : -1;
    const int nbr[8] = {nx0, nx1, ny0, ny1, nz0, nz1, nt0, nt1};
    // Words that can change in this visit: some voxel has room to grow in the
    // word (admissible, not a member) and some voxel or halo holds members of
    // it.  Most tiles carry few of the 8 words' queries; the others are left
    // out of the Jacobi steps (block-uniform).
    {
        uint32_t room = 0, src = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            room |= (a[k] & ~l[k]) ? 1u << k : 0u;
            src |= (l[k] | h[k]) ? 1u << k : 0u;
        }
        __syncthreads();  // the flags were cleared
        if (room) atomicOr(&s_flags[1], room);
        if (src) atomicOr(&s_flags[2], src);
        __syncthreads();
    }
    const uint32_t need = s_flags[1] & s_flags[2];
    // Gauss-Seidel through LDS: the needed words go to LDS once; then each
    // iteration a voxel with room to grow in a word (admissible for a query
    // it is not a member of) ORs its neighbours' current words into it and
    // writes the word back at once if it grew, so a change can travel on
    // within the same iteration (to waves that read after it).  A saturated
    // word cannot change and loads nothing.  Reads racing with writes only
    // see fewer bits (labels only grow); an iteration in which no voxel
    // changed read final values everywhere, which is the local fixed point.
    // The eight words are handled one by one (the register arrays stay in
    // registers only with constant indices).
#define MF4D_STORE_WORD(k) \
    if ((need >> (k)) & 1u) s_lab[(k) * 512 + tid] = l[k];
#define MF4D_STEP_WORD(k)                                                   \
    if (((need >> (k)) & 1u) && (a[k] & ~l[k])) {                          \
        uint32_t nbv = l[k] | h[k];                                         \
        _Pragma("unroll") for (int j = 0; j < 8; ++j)                       \
            if (nbr[j] >= 0) nbv |= s_lab[(k) * 512 + nbr[j]];              \
        const uint32_t sv = nbv & a[k];                                     \
        if (sv != l[k]) {                                                   \
            diff = 1u;                                                      \
            grown = 1u;                                                     \
            l[k] = sv;                                                      \
            s_lab[(k) * 512 + tid] = sv;                                    \
        }                                                                   \
    }
    if (need) {
        MF4D_STORE_WORD(0) MF4D_STORE_WORD(1) MF4D_STORE_WORD(2) MF4D_STORE_WORD(3)
        MF4D_STORE_WORD(4) MF4D_STORE_WORD(5) MF4D_STORE_WORD(6) MF4D_STORE_WORD(7)
        __syncthreads();
        while (true) {
            uint32_t diff = 0;
            MF4D_STEP_WORD(0) MF4D_STEP_WORD(1) MF4D_STEP_WORD(2) MF4D_STEP_WORD(3)
            MF4D_STEP_WORD(4) MF4D_STEP_WORD(5) MF4D_STEP_WORD(6) MF4D_STEP_WORD(7)
            if (!__syncthreads_or(diff != 0)) break;
        }
    }
#undef MF4D_STORE_WORD
#undef MF4D_STEP_WORD
    uint32_t any = 0;
    if (in) {
        any = grown;
        // a tile is swept by one block per phase and nothing else writes its
        // nodes meanwhile (seeds and pushes come in other phases): the node's
        // 32 bytes go back with two plain stores
        if (any) {
            uint4* lp = reinterpret_cast<uint4*>(d.fplanes + v * 8);
            lp[0] = make_uint4(l[0], l[1], l[2], l[3]);
            lp[1] = make_uint4(l[4], l[5], l[6], l[7]);
        }
    }
    if (any) {
        uint32_t faces = 1u << 8;  // bit 8: tile changed
        if (xl == 0) faces |= 1u << 0;
        if (xl == mx) faces |= 1u << 1;
        if (yl == 0) faces |= 1u << 2;
        if (yl == my) faces |= 1u << 3;
        if (zl == 0) faces |= 1u << 4;
        if (zl == mz) faces |= 1u << 5;
        if (tl == 0) faces |= 1u << 6;
        if (tl == mt) faces |= 1u << 7;
        atomicOr(&s_flags[0], faces);
    }
    __syncthreads();
    // lanes 0..7 of the first wave flag the tiles across the eight faces
    // that gained bits
    const uint32_t f = s_flags[0];
    if (f && tid < 8) bschedule_face(d, tile, bx, by, bz, bt, tid, f, par ^ 1);
    // 32 rows of 16 lanes, four to a word
    const uint32_t word = (tid >> 4) & 7;
    if (d.P > 0 && (f || (item.y & kOwn)) && word < (uint32_t)(d.Q + 31) >> 5)
        pull_word(d, tile, word, (tid & 15) + 16 * (tid >> 7), s_ptab);
    __syncthreads();
}

__global__ __launch_bounds__(512) void kb_sweep(DevB d, int par) {
    __shared__ uint32_t s_lab[8 * 512];
    __shared__ uint32_t s_flags[4];
    __shared__ __attribute__((aligned(16))) uint32_t s_ftab[kLdsTab];
    __shared__ __attribute__((aligned(16))) uint32_t s_ptab[kLdsTab];
    __shared__ uint32_t s_pref[kBSubs + 1];
    stage_list(work_counts(d, par), s_pref);
    const uint32_t nwork = s_pref[kBSubs];
    begin_round(d, nwork);
    if (blockIdx.x >= nwork) return;  // block-uniform
    stage_tables(d, 0, s_ftab);
    if (d.P > 0) stage_tables(d, 1, s_ptab);
    __syncthreads();
    for (uint32_t w = blockIdx.x; w < nwork; w += gridDim.x)
        bsweep_tile(d, work_item(d, par, s_pref, w), par, s_lab, s_flags, s_ftab, s_ptab);
}

// L with lane SRC's value (a uniform read) joined into the row ROW of 16 lanes
// where A admits it.
#define MF4D_CROSS(SRC, ROW) \
    L |= (uint32_t)__builtin_amdgcn_readlane((int)L, SRC) & (row == (ROW) ? A0 : 0u);
// A run of admissible steps carries members both ways: inclusive scans over the
// lanes (steps) of (labels, all admissible since), up and then down, within rows
// of 16 lanes by DPP, then across the rows of a group of G lanes.
template <int G>
__device__ __forceinline__ uint32_t spread_up(uint32_t L, uint32_t A0) {
    const int row = lane_id() >> 4;
    uint32_t A = A0;
#define MF4D_UP(CTRL)              \
    {                              \
        L |= dpp<CTRL>(L) & A;     \
        A &= dpp_ones<CTRL>(A);    \
    }
    MF4D_UP(0x111) MF4D_UP(0x112) MF4D_UP(0x114) MF4D_UP(0x118)
#undef MF4D_UP
    A0 = A;
    if (G >= 32) {
        MF4D_CROSS(15, 1)
        if (G == 64) MF4D_CROSS(31, 2)
        MF4D_CROSS(47, 3)
    }
    return L;
}
template <int G>
__device__ __forceinline__ uint32_t spread_down(uint32_t L, uint32_t A0) {
    const int row = lane_id() >> 4;
    uint32_t A = A0;
#define MF4D_DOWN(CTRL)            \
    {                              \
        L |= dpp<CTRL>(L) & A;     \
        A &= dpp_ones<CTRL>(A);    \
    }
    MF4D_DOWN(0x101) MF4D_DOWN(0x102) MF4D_DOWN(0x104) MF4D_DOWN(0x108)
#undef MF4D_DOWN
    A0 = A;
    if (G >= 32) {
        MF4D_CROSS(48, 2)
        if (G == 64) MF4D_CROSS(32, 1)
        MF4D_CROSS(16, 0)
    }
    return L;
}
#undef MF4D_CROSS

// Close and push the particles that gained, a lane per step: G lanes (16, 32 or
// 64, the smallest that hold a trajectory) take a particle, longer trajectories
// go in pieces of 64 steps, up and then down, each piece taking the last lane's
// labels of the one before.  A step that gains queries pushes them into its voxel
// where the voxel is admissible (a plain read of the voxel's labels leaves out
// what it has; the unions need no answer), and marks the voxel.
// Bound by the chain of loads list - labels and ranks - voxels.
// 128^3 x 32, 256 queries, 161,600 visits in 34 rounds: 541 us; 984 with a
// lane per word walking the steps.
template <int G>
__global__ __launch_bounds__(256) void kb_close(DevB d, int par) {
    __shared__ __attribute__((aligned(16))) uint32_t s_ptab[kLdsTab];
    __shared__ __attribute__((aligned(16))) uint32_t s_ftab[kLdsTab];
    __shared__ uint32_t s_pref[kBSubs + 1];
    if (!d.counters[BC_RACT]) return;
    stage_list(d.dcnt, s_pref);
    const uint32_t nd = s_pref[kBSubs];
    if (blockIdx.x == 0 && threadIdx.x == 0) d.stat64[S_PART_VISITS] += nd;
    constexpr uint32_t kPer = 64 / G;  // particles of a wave
    if (blockIdx.x * 4 * kPer >= nd) return;  // block-uniform
    stage_tables(d, 1, s_ptab);
    stage_tables(d, 0, s_ftab);
    __syncthreads();
    const int lane = lane_id(), step = lane & (G - 1);
    const int npar = par ^ 1;
    const int npiece = (d.Tp + G - 1) / G;  // 1 unless G = 64
    const int ndir = d.forward_only ? 1 : 2;
    const int nw = (d.Q + 31) >> 5;
    for (uint32_t i0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * kPer; i0 < nd; i0 += gridDim.x * 4 * kPer) {
        const uint32_t i = i0 + lane / G;
        const bool valid = i < nd;
        uint32_t p = 0;
        if (valid) {
            const int j = sub_list(s_pref, i);
            p = d.dlist[j * d.DCAPB + (i - s_pref[j])];
            if (step == 0) atomicAnd(&d.pdirty[p >> 5], ~(1u << (p & 31)));
        }
        // one piece: up and down at once; more: all up, then all down
        const int nrun = npiece == 1 ? 1 : ndir * npiece;
        uint32_t carry[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int q = 0; q < nrun; ++q) {
            const bool down = q >= npiece;
            if (q == npiece) {
#pragma unroll
                for (int k = 0; k < 8; ++k) carry[k] = 0;
            }
            const int j = (down ? 2 * npiece - 1 - q : q) * G + step;
            const bool have = valid && j < d.Tp;
            uint32_t rank = 0, bin = kNoVoxel;
            uint32_t l[8], n[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) l[k] = 0;
            uint4* lp = reinterpret_cast<uint4*>(d.pplanes + ((uint64_t)j * d.P + p) * 8);
            if (have) {
                rank = d.prank[(uint64_t)p * d.Tpad + j];
                bin = d.bins[(uint64_t)p * d.Tpad + j];
                const uint4 a = lp[0], b = lp[1];
                l[0] = a.x; l[1] = a.y; l[2] = a.z; l[3] = a.w;
                l[4] = b.x; l[5] = b.y; l[6] = b.z; l[7] = b.w;
            }
            uint32_t any = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                n[k] = 0;
                // (carries exist in pieces of 64 only, one particle to a wave)
                if (k < nw && __ballot((l[k] | carry[k]) != 0)) {
                    const uint32_t A = rank_word(s_ptab, rank, k);
                    uint32_t L = l[k];
                    if (npiece == 1) {
                        L = spread_up<G>(L, A);
                        if (ndir == 2) L = spread_down<G>(L, A);
                    } else if (!down) {
                        if (lane == 0) L |= carry[k] & A;
                        L = spread_up<G>(L, A);
                        carry[k] = (uint32_t)__builtin_amdgcn_readlane((int)L, 63);
                    } else {
                        if (lane == 63) L |= carry[k] & A;
                        L = spread_down<G>(L, A);
                        carry[k] = (uint32_t)__builtin_amdgcn_readlane((int)L, 0);
                    }
                    n[k] = L & ~l[k];
                    any |= n[k];
                }
            }
            if (any) {
                lp[0] = make_uint4(l[0] | n[0], l[1] | n[1], l[2] | n[2], l[3] | n[3]);
                lp[1] = make_uint4(l[4] | n[4], l[5] | n[5], l[6] | n[6], l[7] | n[7]);
                if (rank & kCoupled) {
                    int x, y, z, t;
                    bit_to_xyzt(d.g, bin, x, y, z, t);
                    const uint64_t v = vindex(d, x, y, z, t);
                    const uint32_t vr = d.vrank[v];
                    uint32_t* fl = d.fplanes + v * 8;
                    const uint4 a = reinterpret_cast<const uint4*>(fl)[0], b = reinterpret_cast<const uint4*>(fl)[1];
                    const uint32_t have8[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
                    uint32_t pushed = 0;
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const uint32_t pw = n[k] ? n[k] & ~have8[k] & rank_word(s_ftab, vr, k) : 0u;
                        if (pw) atomicOr(&fl[k], pw);
                        pushed |= pw;
                    }
                    if (pushed) bmark_voxel(d, x, y, z, t, npar);
                }
            }
            // the pieces of the way down read what the way up wrote
            if (npiece > 1) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        }
    }
}

// The work list (tile, flags) of the round of parity `par` from the tiles flagged for it
// (the flags cleared for that parity's next use): a flagged tile joins if it
// holds a node admissible for some query.  Appends go to sub-list (tile mod
// kBSubs): 64 counters on separate lines.  The lists that the round before has
// worked off are emptied.  first: after seeding; also gives every tile its range
// of the coupled list (its end, which kb_couple counts down).
__global__ __launch_bounds__(256) void kb_compact(DevB d, int par, int first) {
    if (!first && !d.counters[BC_RACT]) return;
    if (blockIdx.x == 0 && threadIdx.x < kBSubs) {
        d.wcnt[((uint32_t)(par ^ 1) * kBSubs + threadIdx.x) * kBCntStride] = 0u;
        d.dcnt[threadIdx.x * kBCntStride] = 0u;
    }
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i0 = blockIdx.x * blockDim.x; i0 < d.NTB; i0 += stride) {  // block-uniform
        const uint32_t i = i0 + threadIdx.x;
        if (i < d.NTB) {
            uint32_t* f = &d.dirty[(size_t)par * d.NTB + i];
            const uint32_t bits = *f;
            if (bits) {
                *f = 0u;
                if (d.active[i]) {
                    const uint32_t j = (uint32_t)par * kBSubs + (i & (kBSubs - 1));
                    const uint32_t k = atomicAdd(&d.wcnt[j * kBCntStride], 1u);
                    d.work[(size_t)j * d.WCAPB + k] = make_uint2(i, bits);
                }
            }
        }
        if (first && d.P > 0) {
            uint32_t x = i < d.NTB ? d.tcnt[i] : 0u;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(x, o);
                if (lane_id() >= o) x += y;
            }
            uint32_t base = 0;
            if (lane_id() == 63 && x) base = atomicAdd(&d.counters[BC_NLIST], x);
            base = __shfl(base, 63);
            if (i < d.NTB) d.tbase[i] = base + x;
        }
    }
}

// The end of a chunk of rounds for the host, one wave: the work lists' lengths,
// the counters and the statistics into pinned memory, then the sequence number the
// host polls.  The count of rounds starts again at 0.
__global__ void kb_report(DevB d, unsigned long long* host, uint32_t* host_counters, uint32_t* host_seq,
                          uint32_t seq) {
    const int lane = threadIdx.x;
    for (int par = 0; par < 2; ++par) {
        uint32_t x = work_counts(d, par)[lane * kBCntStride];
        for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
        if (lane == 0) host_counters[BC_NWORK0 + par] = x;
    }
    if (lane > BC_NWORK1 && lane < BC_NCOUNTERS) host_counters[lane] = d.counters[lane];
    if (lane < S_NSTAT) host[lane] = d.stat64[lane];
    if (lane == BC_ROUNDS) d.counters[BC_ROUNDS] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
    if (lane == 0) __hip_atomic_store(host_seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void kb_reset(DevB d) {
    const uint64_t tid = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = tid; i < 2ull * d.NTB; i += stride) d.dirty[i] = 0;
    for (uint64_t i = tid; i < d.NTB; i += stride) d.tcnt[i] = 0;
    for (uint64_t i = tid; i < ((uint64_t)d.NTB + 3) / 4; i += stride)
        reinterpret_cast<uint32_t*>(d.active)[i] = 0;
    for (uint64_t i = tid; i < (uint64_t)(d.P + 31) / 32; i += stride) d.pdirty[i] = 0;
    if (tid < BC_NCOUNTERS) d.counters[tid] = 0;
    if (tid < 2 * kBSubs) d.wcnt[tid * kBCntStride] = 0;
    if (tid < kBSubs) d.dcnt[tid * kBCntStride] = 0;
    if (tid < S_NSTAT) d.stat64[tid] = 0;
}

inline unsigned grid_for(uint64_t n, unsigned block, unsigned cap) {
    uint64_t b = (n + block - 1) / block;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

}  // namespace

void launch_b_prepare(const DevB& d, const int32_t* seeds, int64_t S, hipStream_t s) {
    const uint64_t V = (uint64_t)d.X * d.Y * d.Z * d.T;
    const uint64_t n = (uint64_t)d.P * d.Tpad;
    hipLaunchKernelGGL(kb_reset, dim3(grid_for(2ull * d.NTB + d.P / 32 + 1, 256, 2048)), dim3(256),
                       0, s, d);
    hipLaunchKernelGGL(kb_admit_field, dim3(grid_for(V, 1024, 4096)), dim3(256), 0, s, d);
    if (d.P > 0) hipLaunchKernelGGL(kb_admit_particles, dim3(grid_for(n, 1024, 8192)), dim3(256), 0, s, d);
    if (S > 0)
        hipLaunchKernelGGL(kb_seeds, dim3(grid_for(S, 256, 1u << 20)), dim3(256), 0, s, d, seeds, S);
    hipLaunchKernelGGL(kb_compact, dim3(grid_for(d.NTB, 256, 1024)), dim3(256), 0, s, d, 0, 1);
    if (d.P > 0) hipLaunchKernelGGL(kb_couple, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, d);
}

namespace {
template <int LX, int LY, int LZ, int LT>
void sweep_shape(const DevB& d, int par, hipStream_t s) {
    hipLaunchKernelGGL((kb_sweep_tiles<LX, LY, LZ, LT>), dim3(grid_for((uint64_t)d.NTB * ((d.Q + 127) / 128), 4, 1024)),
                       dim3(256), 0, s, d, par);
}
}  // namespace

void launch_b_round(const DevB& d, uint32_t round, hipStream_t s) {
    const int par = round & 1;
    // the shapes of at least 4 x 4 nodes along x and y that the search over tile
    // shapes tries; any other goes through LDS
    switch (d.lx * 1000 + d.ly * 100 + d.lz * 10 + d.lt) {
        case 2223: sweep_shape<2, 2, 2, 3>(d, par, s); break;
        case 3222: sweep_shape<3, 2, 2, 2>(d, par, s); break;
        case 3330: sweep_shape<3, 3, 3, 0>(d, par, s); break;
        case 3321: sweep_shape<3, 3, 2, 1>(d, par, s); break;
        case 4221: sweep_shape<4, 2, 2, 1>(d, par, s); break;
        case 4320: sweep_shape<4, 3, 2, 0>(d, par, s); break;
        case 5220: sweep_shape<5, 2, 2, 0>(d, par, s); break;
        case 2322: sweep_shape<2, 3, 2, 2>(d, par, s); break;
        default: hipLaunchKernelGGL(kb_sweep, dim3(grid_for(d.NTB, 1, 2048)), dim3(512), 0, s, d, par); break;
    }
    if (d.P > 0) {
        const int G = d.Tp <= 16 ? 16 : d.Tp <= 32 ? 32 : 64;
        const dim3 close(grid_for((uint64_t)d.P, 4 * (64 / G), 1024));
        if (G == 16) hipLaunchKernelGGL(kb_close<16>, close, dim3(256), 0, s, d, par);
        else if (G == 32) hipLaunchKernelGGL(kb_close<32>, close, dim3(256), 0, s, d, par);
        else hipLaunchKernelGGL(kb_close<64>, close, dim3(256), 0, s, d, par);
    }
    hipLaunchKernelGGL(kb_compact, dim3(grid_for(d.NTB, 256, 1024)), dim3(256), 0, s, d, par ^ 1, 0);
}

void launch_b_report(const DevB& d, unsigned long long* host, uint32_t* host_counters, uint32_t* host_seq,
                     uint32_t seq, hipStream_t s) {
    hipLaunchKernelGGL(kb_report, dim3(1), dim3(64), 0, s, d, host, host_counters, host_seq, seq);
}

}  // namespace mf4d
