// Host-side launchers of the device kernels (defined in cashash_kernels.hip).
#pragma once
#include "cashash_internal.h"

namespace cashash {
hipError_t launch_fill_u64(hipStream_t s, unsigned long long* p, int64_t n, unsigned long long v);
hipError_t launch_fill_u32(hipStream_t s, uint32_t* p, int64_t n, uint32_t v);
hipError_t launch_colsum(hipStream_t s, const ImgDev* imgs, const RowChunk* chunks, int n_chunks,
                         unsigned long long* S);
// Column sums of a whole set in one launch, with what follows from them: the
// bias.  S: kSumWords words, the first kSumClear zero, the totals from
// kSumTotal on afterwards; next_S (cleared the same way for the next call) and
// the recompute counts are cleared.
hipError_t launch_colsum_bias(hipStream_t s, const ImgDev* imgs, const RowChunk* chunks, int n_chunks,
                              unsigned long long* S, const double* Rt, double n_tot, float* bias,
                              unsigned long long* next_S, unsigned long long* counts);
hipError_t launch_bias(hipStream_t s, const double* Rt, const unsigned long long* S, double n_tot, float* bias);
// Projection with the binary64 recompute of what falls inside the margin; the
// number of recomputes is added to counts.  near: pl.near_bytes() bytes.
hipError_t launch_proj_mfma(hipStream_t s, const ImgDev* imgs, const CodeOut* outs, const RowChunk* tiles, int n_tiles,
                            const uint4* frag, const float* bias, float margin, const double* R,
                            const unsigned long long* S, double n_tot, unsigned long long* counts, const ProjPlan& pl,
                            void* near);
hipError_t launch_proj_fp32(hipStream_t s, const ImgDev* imgs, const CodeOut* outs, const RowChunk* tiles, int n_tiles,
                            const float* R32, const float* bias, float margin, const double* R,
                            const unsigned long long* S, double n_tot, unsigned long long* counts, const ProjPlan& pl,
                            void* near);
// Work items of the pair tile table; clears the call's control words.
hipError_t launch_make_items(hipStream_t s, const ItemArgs& a, const ImgDev* imgs);
// The bucket tables of the train images and, with items, the work items too.
hipError_t launch_bucket(hipStream_t s, bool epi, const ImgDev* imgs, const TableOut* touts,
                         const int32_t* train_list, int n_train, const ItemArgs* items);
// One matcher launch over items [0, n_items), or the same as a node of a graph.
struct MatchLaunch {
    bool epi;
    int ns, grid;
    const ImgDev* imgs;
    const PairDev* pairs;
    const Item* items;
    int32_t n_items;
    uint32_t* ctl;
    MatchParams prm;
    int32_t *o_idx, *o_d1, *o_d2;
};
hipError_t launch_match(hipStream_t s, const MatchLaunch& L);
hipError_t add_match_node(hipGraph_t graph, hipGraphNode_t* node, const hipGraphNode_t* after, const MatchLaunch& L);
}  // namespace cashash

// Geometry-aware first stage (defined in cashash_geometry.hip).
namespace cashash {
hipError_t launch_top_scale(hipStream_t s, const SelectImg* imgs, int n_images);
hipError_t launch_gather_rows(hipStream_t s, const GatherImg* imgs, const RowChunk* chunks, int n_chunks,
                              unsigned* err);
size_t fundamental_lds_bytes(int cap);
hipError_t launch_fundamental(hipStream_t s, const GeoImg* imgs, const GeoPair* pairs, int64_t n_pairs,
                              const int32_t* match_idx, const uint32_t* rnd, const GeoParams& prm, const GeoOut& out,
                              GeoFit* fits, unsigned* err);
}  // namespace cashash
