// Device-side data layouts shared by the host runtime and the kernels of the
// CasHash matcher (gfx950).  Nothing here is part of the public C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cashash {

constexpr int kDim = 128;          // SIFT dimension d
constexpr int kTables = 6;         // lookup tables (Step 1)
constexpr int kKeyBits = 8;        // m bits per lookup key
constexpr int kCodeBits = 128;     // n bits of the remapping code (Step 2)
constexpr int kRows = kCodeBits + kTables * kKeyBits;  // 176 projection rows
constexpr int kRowTiles = kRows / 16;                   // 11 MFMA row tiles
constexpr int kOffStride = 257;    // bucket offsets per table (256 keys + end)
constexpr int kMaxK = 64;
constexpr int kSelCap = 384;       // per-wave LDS list of a query tile's kept candidates
// The plain matcher finds a candidate's bucket run by masks of run starts for
// the first 64 x `slots` candidates of a query (4 or 8, a template parameter);
// a query with more takes compares for the rest.  Pairs run 4 up to kLargeTrain
// train points (expected candidates per query: about 0.0255 per train point,
// 230 at 9000) and 8 above: fewer masks, less LDS and one more block per CU.
constexpr int kLargeTrain = 9000;
constexpr int kWavesPerBlock = 4;  // matcher block = 4 waves
constexpr int kMaxTile = 32;       // queries per matcher work item (one per lane of the tile setup)
constexpr int kBucketWaves = 8;    // wavefronts per (train image, table) counting sort
constexpr int kProjTB = 4;         // 16-descriptor tiles per projection block

// Per-image view.  desc/codes/keys/kp are the caller's (or staged) buffers;
// off/ent are the bucket tables the library builds for train images.
struct ImgDev {
    const uint8_t* desc;   // [n][128]
    const uint64_t* codes; // [n][2]
    const uint8_t* keys;   // [n][6]
    const float* kp;       // [n][2] or null
    const uint32_t* off;   // [6][257] bucket start offsets, or null
    const uint8_t* ent;    // [6][n] bucket-ordered entries, or null
    int32_t n;
    int32_t pad;
};

// Writable per-image outputs of the code builder.
struct CodeOut {
    uint64_t* codes;   // [n][2]
    uint8_t* keys;     // [n][6]
    int64_t pad;
};

// A 64-projection word of a descriptor with at least one projection inside the
// rounding margin: image, row and the mask of what to recompute in binary64.
struct NearEntry {
    int32_t img;
    int32_t row;
    uint32_t mask[2];
};
constexpr int kNearSegs = 2;       // projection blocks per recompute block and word
constexpr int kNearThreads = 512;

// How the projection of n_tiles tiles of 16 descriptors is cut: groups of tpg
// tiles, `grid` blocks taking groups a grid apart.
struct ProjPlan {
    int tpg, groups, grid;
    bool fused;  // one group per block, recomputed by the block
    uint32_t seg_cap() const { return (uint32_t)((groups + grid - 1) / grid) * (uint32_t)tpg * 16u; }
    size_t count_bytes() const { return ((size_t)grid * 12 + 255) & ~size_t(255); }
    size_t near_bytes() const { return fused ? 0 : count_bytes() + (size_t)grid * 3 * seg_cap() * sizeof(NearEntry); }
};

// Two blocks fit on a compute unit (R in registers).  Fewer tiles than that
// many groups of kProjTB: smaller groups on all of them, and the block
// recomputes its own margin hits (a launch less: 32000 descriptors
// 43.3 us per call against 48.1, 8000 37.3 against 39.8).
inline ProjPlan proj_plan(int n_tiles, int n_cu) {
    const int blocks = 2 * n_cu;
    ProjPlan p;
    p.fused = n_tiles <= blocks * kProjTB;
    p.tpg = p.fused ? (n_tiles + blocks - 1) / blocks : kProjTB;
    if (p.tpg < 1) p.tpg = 1;
    p.groups = (n_tiles + p.tpg - 1) / p.tpg;
    p.grid = p.groups < blocks ? p.groups : blocks;
    return p;
}

// The plain FP32 form: a block per 16 tiles (a thread per descriptor), always
// with the near list.
inline ProjPlan plain_plan(int n_tiles) {
    ProjPlan p;
    p.tpg = 16;
    p.groups = p.grid = (n_tiles + 15) / 16;
    p.fused = false;
    return p;
}

// Column sums of a whole set: kSumSlots copies of kDim sums, the ticket of the
// blocks that added to them, and the totals.  Sums over several launches use
// the first kDim words alone.
constexpr int kSumSlots = 8;
constexpr int kSumClear = kSumSlots * kDim + 1;
constexpr int kSumTotal = kSumSlots * kDim + 8;
constexpr int kSumWords = kSumTotal + kDim;
// Counters of recomputed projections, one of kCountSlots per block, a 64-byte
// line apart.
constexpr int kCountSlots = 64;
constexpr int kCountStride = 8;
constexpr int kCountWords = kCountSlots * kCountStride;

// Writable bucket tables of one train image.
struct TableOut {
    uint32_t* off;     // [6][257]
    uint8_t* ent;      // bucket-ordered entries, ent_bytes(n, epi)
};

// Bucket-ordered entries of a train image, struct of arrays over the six
// tables: for table t and position s (entries of one bucket contiguous, in
// ascending index order)
//   code[t][s] : the point's 128-bit code (16 B)
//   kid[t][s]  : keys and index as the matcher's union test takes them (8 B,
//                entry_word)
//   kp[t][s]   : its keypoint (epipolar form only)
// laid out one after another from TableOut::ent / ImgDev::ent.
inline __host__ __device__ size_t ent_bytes(int n, bool epi) { return (size_t)kTables * n * (epi ? 32 : 24); }

struct PairDev {
    int32_t qi, ti;     // query image, train image
    int64_t out;        // first output slot of this pair
    double F[9];        // row-major fundamental matrix (epipolar form)
};

struct Item {           // a tile of consecutive queries of one pair (nq <= kMaxTile, nq * k <= kSelCap)
    int32_t pair;
    int32_t q0;
    int32_t nq;
    int32_t pad;
};

struct PairTiles {      // pair `pair`'s query tiles are items [first, first + count)
    int32_t pair;
    int32_t first;
};

struct RowChunk {       // rows [r0, r0 + nr) of image img
    int32_t img;
    int32_t r0;
    int32_t nr;
    int32_t pad;
};

// Resident blocks per compute unit the matcher kernels are compiled for, and
// their persistent launches use (LDS per block: 18.6 KB, 22.7 KB in the 8-slot
// form, 20.6 KB in the band form; 8 blocks leave 64 registers, 7 leave 72).
// 60 x 8000 points: 4 blocks 5.8 ms, 6 4.9, 7 4.53, 8 4.40; 40 x 12000 (8
// slots): 6 blocks 4.29 ms, 7 4.06.
constexpr int match_blocks_per_cu(bool epi, int ns) { return epi || ns > 4 ? 7 : 8; }

constexpr int kSegments = 8;       // one work segment per XCD
// Control words of a matcher call: a line of kCtlStride words per segment
// holds its work counter (one per launch of the call) and kStatsPerLine places
// for statistics.
constexpr int kCtlStride = 64;
constexpr int kCtlWords = kSegments * kCtlStride;
constexpr int kStatsPerLine = 3;
constexpr int kStatSlots = kSegments * kStatsPerLine;
inline __host__ __device__ unsigned long long* stat_slot(uint32_t* ctl, int i) {
    return reinterpret_cast<unsigned long long*>(ctl + (i % kSegments) * kCtlStride + 16 * (1 + i / kSegments));
}

// What the work items of a match call are made of.
struct ItemArgs {
    const PairTiles* pt;
    const PairDev* pairs;
    Item* items;
    uint32_t* ctl;
    int32_t n_pt, qt, n_items, pad;
};

struct MatchParams {
    int32_t k;
    int32_t tau;
    int64_t num2;       // ratio_num^2
    int64_t den2;       // ratio_den^2
    double max_px;
    // persistent scheduling (grab > 0): items [seg[x], seg[x+1]) are segment x,
    // handed out `grab` at a time, by counter `set` of its control line; a wave
    // starts on its own XCD's segment and moves to the others when it is
    // exhausted.  grab == 0: wavefront w of the grid takes item w only.
    int32_t seg[kSegments + 1];
    int32_t grab;
    int32_t set;
};

// Bf16 hi/lo fragments of the 176 projection rows, pre-arranged so that lane
// l of a wave loads its 8 values for (part, row tile, k step) as one 16-byte
// vector: frag[part][rt][ks][l][i] = part(R[16 rt + l % 16][32 ks + 8 (l / 16) + i]).
constexpr int kFragBytes = 2 * kRowTiles * 4 * 64 * 16;

// ---- geometry-aware first stage (Sec. 3.1) ---------------------------------

// Top-scale selection of one image: rows_out[0..m) receives the m largest
// scales' indices in ascending index order.
struct SelectImg {
    const float* scale;  // [n]
    int32_t* rows_out;   // [m]
    int32_t n, m;
};

// Row gather of one image: out row j = in row rows[j]; a null output pointer
// skips that field.
struct GatherImg {
    const uint8_t* desc;    // [n][128]
    const uint64_t* codes;  // [n][2]
    const uint8_t* keys;    // [n][6]
    const float* kp;        // [n][2]
    const int32_t* rows;    // [m]
    uint8_t* o_desc;
    uint64_t* o_codes;
    uint8_t* o_keys;
    float* o_kp;
    int32_t n, m;
};

// Keypoints of an image the stage-1 matches index.
struct GeoImg {
    const float* kp;  // [n][2]
    int32_t n;
    int32_t pad;
};

struct GeoPair {
    int32_t qi, ti;
    int64_t out;      // first stage-1 output slot of the pair (n of qi slots)
};

struct GeoParams {
    int32_t n_hyp;        // hypotheses (rows of the 8-draw table)
    int32_t min_matches;  // fewer stage-1 matches: not estimated
    double thr;           // inlier distance to the epipolar line, px
    int32_t cap;          // matches held in LDS per pair (>= every pair's query count)
    int32_t pad;
};

struct GeoOut {
    double* F;            // [P][9]
    int32_t* n_matches;   // [P]
    int32_t* n_inliers;   // [P]
    int32_t* best_h;      // [P]
    int32_t* status;      // [P]
};

// What the fit of a pair leaves for its refit: A^T A of the best hypothesis's
// inliers and the two normalisations (query s, cx, cy, then train); refit == 0
// if the pair's outputs are final already.
struct GeoFit {
    double A[81];
    double norm[6];
    int32_t refit;
    int32_t pad;
};
constexpr size_t kGeoRowBytes = 256 * 9 * sizeof(double);  // LDS of one chunk's design rows

constexpr int kGeoMaxMatches = 8192;  // LDS list of one pair's stage-1 matches (16 B each)
constexpr int kJacobiSweeps3 = 6;
constexpr int kJacobiSweeps9 = 10;

}  // namespace cashash
