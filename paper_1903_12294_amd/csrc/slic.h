// Internal declarations of the 4D SLIC clustering kernels (slic.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mf4d_internal.h"

namespace mf4d {

// Accumulators of one centre: quantised sums (x, y, z, t, point value, field
// value) and the counts of field and point samples, as 64-bit integers.
enum SlicAcc : int { SA_X = 0, SA_Y, SA_Z, SA_T, SA_P, SA_F, SA_NF, SA_NP, kSlicAcc = 8 };

// Copies of the centres' sums, among which the blocks spread their additions: up to
// eight while they are few (the update reads them all: 1 us more for 128 centres
// in eight copies).  35 x 28 x 10 x 44, 6 centres: 16 us a pass, 58 with one copy.
constexpr int slic_copies(int64_t K) { return K <= 32 ? 8 : K <= 64 ? 4 : K <= 128 ? 2 : 1; }

// Device counters of a run.
enum SlicCounter : int {
    SC_MOVED = 0,   // centres whose values changed by more than eps this update
    SC_RANGE = 1,   // a value outside |v| < 2048 was met (quantised sums could overflow)
    SC_ITERS = 2,   // assignment passes done
    SC_DONE = 3,    // nothing moved, or out of range: passes still queued do nothing
    SC_TICKET = 4,  // blocks of the update that have finished
    kSlicCounters = 8
};

struct DevS {
    int X, Y, Z, T;
    int64_t P;
    int Tp;              // particle steps (point sample tau at time tau / r)
    int k[4];            // centres per axis (x, y, z, t)
    int K;               // k[0] * k[1] * k[2] * k[3]
    float C[4];          // grid intervals E_d / k_d (fp32)
    float wd, wf, wp, cf;
    double eps;
    const float* field;  // [T][Z][Y][X]
    const float4* spos;  // [Tp * P]: point samples in visiting order, (x, y, z, t)
    const float* sattr;  // [Tp * P]: their values, same order
    int32_t* labels;     // [V + Tp * P]: field samples [T][Z][Y][X], then point samples in
                         // visiting order
    unsigned long long* acc;  // [copies][K][kSlicAcc]
    int copies;               // of the sums, a power of two (slic_copies)
    double* cen;         // [K][6]: x, y, z, t, p, f
    float* cen32;        // [K][8]: the same rounded to fp32, then 2 unused
    long long* cnt;      // [K][2]: field and point samples of each centre
    // Per axis d and seed-grid slab i (centres with cell index i on axis d):
    // the least and greatest centre coordinate, as order-preserving keys,
    // at [(0 * 4 + d) * kmax + i] (least) and [(1 * 4 + d) * kmax + i].
    // Two buffers: the passes read slab, the update that ends them fills slab_next.
    uint32_t *slab, *slab_next;
    // Per axis d and seed cell j: the least and greatest slab index whose
    // centres can reach a sample of cell j, at [(d * kmax + j) * 2] and + 1
    // (empty: least > greatest).
    int* reach;
    int mask_slabs;      // widest reach range searched through bit masks (0..32); wider ranges
                         // take the general loop
    int boxes;           // candidate lists per box of samples (0: every sample on its own)
    float tie;           // distances this close (w_d 1e-18) are compared again with denormals scaled
    int kmax;            // max(k[0..3])
    uint32_t* counters;  // SlicCounter
    uint32_t* host;      // pinned host memory: SC_RANGE, SC_ITERS, SC_DONE after each update
    uint32_t* over;      // boxes whose list did not fit: their number, then slic_boxes() entries
    unsigned long long* lsum;  // [K][kSlicAcc]: the sums of the last update (for the features)
};

// Cluster merging and feature statistics (Section 3.3).  Feature ids are
// centre ids (the lowest of each merged group).
enum FeatStat : int {
    FS_NF = 0, FS_NP, FS_MEAN_F, FS_MEAN_P, FS_STD_F, FS_STD_P,
    FS_XMIN, FS_XMAX, FS_YMIN, FS_YMAX, FS_ZMIN, FS_ZMAX, FS_TMIN, FS_TMAX, kFeatStats
};

struct DevM {
    int K;
    double eps;
    int* parent;             // [K] union-find links
    int32_t* feat;           // [K] feature of each centre (-1: no samples)
    unsigned long long* fsum;  // [K][kSlicAcc] integer sums per feature
    double* fmean;           // [K][2] mean field, point value per feature
    uint32_t* cext;          // [K][8] per centre: least x, y, z, t keys, then greatest
    double* css;             // [K][2] per centre: squared deviations from its feature's means
    uint32_t* fext;          // [K][8] per feature, the same
    double* fss;             // [K][2] per feature
    double* out;             // [K][kFeatStats]
    uint32_t* err;           // set if a union-find wait ran out (never expected)
};

// Merge the centres of the last run (labels, centres, counts, sums in s) and
// compute the features' statistics into m.out.  Errors as a HIP result.
int launch_slic_merge(const DevS& s, const DevM& m, hipStream_t st);

// Visiting order of the point samples: particle-steps sorted by the sub-box (8 x
// 4 x 4 x 4 voxel-steps) holding them, tile by tile, steps in no voxel last;
// order[t * P + p] = the position of that step in the visiting order.  Their
// positions and times (spos; time t / r in field steps, r particle steps per
// field step) and values (sattr) are copied in that order from xyz [T][P][3]
// and attr [T][P] (T particle steps).  bins: [P][Tpad] voxel bits of tiles with
// 2^logBT steps (~0u: none); scratch: slic_order_keys() + 1 + 1024 words.  Errors
// as a HIP result.
inline uint32_t slic_order_keys(uint32_t ntiles, int logBT) { return (ntiles << (2 + logBT)) + 1; }
int launch_slic_order(const uint32_t* bins, const float* xyz, const float* attr, int64_t P, int Tpad,
                      int T, int r, int logBT, uint32_t ntiles, uint32_t* scratch, uint32_t* order,
                      float4* spos, float* sattr, hipStream_t st);
// Point labels from visiting order back to [T][P]: out[q] = in[order[q]]
// (order as written by launch_slic_order).
void launch_slic_unsort(const int32_t* in, const uint32_t* order, int T, int64_t P, int32_t* out, hipStream_t st);
// Trajectory segments (Section 3.4), in place on point labels [T][P]: the
// feature id (feat[label]) where the particle has that feature at t - 1 or
// t + 1, else -1.
void launch_slic_segments(int32_t* lab, const int32_t* feat, int T, int64_t P, hipStream_t st);
// Boxes of samples a pass takes (field boxes and point blocks).
uint32_t slic_boxes(const DevS& s);
// Start of a run: sums and counters cleared, labels from the seed cells, their
// sums, and the first centres (with slab bounds in s.slab_next).
void launch_slic_begin(const DevS& s, hipStream_t st);
// One iteration: an assignment pass over both sample types with the sums of the
// new labels, then the centres from the sums (the sums cleared), compared with
// the previous ones, and the slab bounds of the new centres.  Does nothing once
// SC_DONE is set, so that iterations can be queued ahead of the host.
void launch_slic_iteration(const DevS& s, hipStream_t st);

}  // namespace mf4d
