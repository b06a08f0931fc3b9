// HIP kernels of the hash-code and bucket-table steps for gfx950 (MI355X).
//
// Hash codes ("The Improved Parallel Calculation of Hashing Code"): the
// paper's one-block-per-(point, bit) reduction is replaced by a dense
// contraction on the matrix cores: descriptors (uint8, exact in bf16) times
// the projection rows split into bf16 hi + lo parts, fp32 accumulate.  A
// projection whose value lies within a proven rounding margin of zero is
// recomputed in binary64 exactly as the reference definition does it.
// Bucket tables: per train image and table, a stable counting sort of the
// 8-bit keys whose entries carry code, keys and index (Step 1 lookup runs).
#include <algorithm>

#include "cashash_device.h"

namespace cashash {

// ------------------------------------------------------------------ utilities

__global__ void fill_u64_kernel(unsigned long long* p, int64_t n, unsigned long long v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void fill_u32_kernel(uint32_t* p, int64_t n, uint32_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Work items from the per-pair tile table: item i belongs to the last entry
// whose first tile is <= i (binary search); its queries are tile (i - first)
// of that pair's query image, qt per tile.  Also clears the matcher's control
// words.
__device__ __forceinline__ void make_item(const ItemArgs& a, const ImgDev* __restrict__ imgs, int32_t i) {
    if (i < kCtlWords) a.ctl[i] = 0u;
    if (i >= a.n_items) return;
    int32_t lo = 0, hi = a.n_pt - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (a.pt[mid].first <= i) lo = mid; else hi = mid - 1;
    }
    const int32_t p = a.pt[lo].pair;
    const int32_t q0 = (i - a.pt[lo].first) * a.qt;
    const int32_t nq = imgs[a.pairs[p].qi].n;
    a.items[i] = Item{p, q0, min(a.qt, nq - q0), 0};
}

__global__ void make_items_kernel(ItemArgs a, const ImgDev* __restrict__ imgs) {
    make_item(a, imgs, (int32_t)(blockIdx.x * blockDim.x + threadIdx.x));
}

// ------------------------------------------------------------------ column sums
// bias_j = (r_j . S) / N in binary64, rounded once to fp32 for the fast path.
// One block of at least kRows threads; Rt is R transposed ([128][kRows]: a
// component's values side by side), s_S the sums in LDS.
__device__ __forceinline__ void bias_block(const double* __restrict__ Rt, const double* s_S, double n_tot,
                                           float* __restrict__ bias) {
    const int j = threadIdx.x;
    if (j >= kRows) return;
    double acc = 0.0;
#pragma unroll 32
    for (int i = 0; i < kDim; ++i) acc = fma(Rt[i * kRows + j], s_S[i], acc);
    bias[j] = (float)(acc / n_tot);
}

// One block per chunk of rows.  Thread t reads the 16-byte column group t % 8
// of rows t / 8, t / 8 + 32, ...; partial column totals meet in LDS and each
// column is added to the int64 sums with one atomic.
// WHOLE: the grid covers the whole set.  The blocks add to one of kSumSlots
// copies of the sums (one copy's 128 addresses would queue every block's
// atomics); the last block to finish (a ticket after its sums) adds the copies
// up, sets the bias, and clears the copies that the next call will use and the
// recompute counts, so that none of it needs a launch.  An atomic's returned
// value is the proof that it took place, which is all that the ticket must
// follow: a fence here would write the caches back once per wavefront (800k
// descriptors: 56 us with it).
// Bound by the read and by the adds at its end: 800k descriptors 24.9 us, 4.1
// TB/s (29 + 7 us with the bias a launch of its own).
template <bool WHOLE>
__global__ __launch_bounds__(256) void colsum_kernel(const ImgDev* __restrict__ imgs,
                                                     const RowChunk* __restrict__ chunks,
                                                     unsigned long long* __restrict__ S, const double* __restrict__ Rt,
                                                     double n_tot, float* __restrict__ bias,
                                                     unsigned long long* __restrict__ next_S,
                                                     unsigned long long* __restrict__ counts) {
    __shared__ uint32_t part[32][kDim + 1];
    __shared__ double s_S[kDim];
    __shared__ uint32_t s_last;
    const RowChunk ch = chunks[blockIdx.x];
    const uint8_t* base = imgs[ch.img].desc + (int64_t)ch.r0 * kDim;
    const int g = threadIdx.x & 7, rl = threadIdx.x >> 3;
    uint32_t s[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) s[c] = 0;
#pragma unroll 8
    for (int r = rl; r < ch.nr; r += 32) {
        const uint4 w = gload(reinterpret_cast<const uint4*>(base + (int64_t)r * kDim + g * 16));
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) s[a * 4 + b] += (ws[a] >> (8 * b)) & 0xFFu;
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) part[rl][g * 16 + c] = s[c];
    __syncthreads();
    unsigned long long* to = S + (WHOLE ? (blockIdx.x % kSumSlots) * kDim : 0);
    if (threadIdx.x < kDim) {
        uint32_t tot = 0;
        for (int r = 0; r < 32; ++r) tot += part[r][threadIdx.x];
        const unsigned long long old = atomicAdd(&to[threadIdx.x], (unsigned long long)tot);
        if constexpr (WHOLE) asm volatile("" ::"v"(old) : "memory");
    }
    if constexpr (WHOLE) {
        __syncthreads();
        unsigned long long* ticket = S + kSumSlots * kDim;
        if (threadIdx.x == 0) s_last = atomicAdd(ticket, 1ull) + 1ull == (unsigned long long)gridDim.x;
        __syncthreads();
        if (!s_last) return;
        if (threadIdx.x < kDim) {
            unsigned long long tot = 0, v[kSumSlots];
#pragma unroll
            for (int q = 0; q < kSumSlots; ++q) v[q] = atomicAdd(&S[q * kDim + threadIdx.x], 0ull);
#pragma unroll
            for (int q = 0; q < kSumSlots; ++q) tot += v[q];
            S[kSumTotal + threadIdx.x] = tot;
            s_S[threadIdx.x] = (double)tot;
        }
        for (int i = threadIdx.x; i <= kSumSlots * kDim; i += 256) next_S[i] = 0ull;
        for (int i = threadIdx.x; i < kCountWords; i += 256) counts[i] = 0ull;
        __syncthreads();
        bias_block(Rt, s_S, n_tot, bias);
    }
}

// The bias alone, of sums added up over several launches.
__global__ __launch_bounds__(256) void bias_kernel(const double* __restrict__ Rt,
                                                   const unsigned long long* __restrict__ S, double n_tot,
                                                   float* __restrict__ bias) {
    __shared__ double s_S[kDim];
    if (threadIdx.x < kDim) s_S[threadIdx.x] = (double)S[threadIdx.x];
    __syncthreads();
    bias_block(Rt, s_S, n_tot, bias);
}

// ------------------------------------------------------------------ projection
__device__ __forceinline__ uint32_t bf16_pair(uint32_t w, int sh) {
    const float f0 = (float)((w >> sh) & 0xFFu);
    const float f1 = (float)((w >> (sh + 8)) & 0xFFu);
    return (__float_as_uint(f0) >> 16) | (__float_as_uint(f1) & 0xFFFF0000u);
}

__device__ __forceinline__ bf16x8 load_frag(const uint4* __restrict__ frag, int idx) {
    union {
        uint4 u;
        bf16x8 v;
    } cv;
    cv.u = frag[idx];
    return cv.v;
}

// ---- binary64 recompute
// Near-margin projections are recomputed with the same fused multiply-add
// chain over components 0..127 of r_j . (N x - S) that defines the codes
// (N x_i - S_i is an exact integer in binary64), row rp per lane (vector loads,
// 16 components at a time).
// Each group of 16 is loaded while the one before it is multiplied.
__device__ __forceinline__ double near_chain(const uint8_t* x, const double* rp, const double* s_S, double n_tot) {
    const uint4* xp = reinterpret_cast<const uint4*>(x);
    const double2* rr = reinterpret_cast<const double2*>(rp);
    double2 rv[2][8];
    uint4 xv[2];
    auto fetch = [&](int h, int q) {
        xv[h] = gload(xp + q);
#pragma unroll
        for (int i = 0; i < 8; ++i) rv[h][i] = rr[8 * q + i];
        __builtin_amdgcn_sched_barrier(0);
    };
    double p = 0.0;
    auto chain = [&](int h, int q) {
        const uint32_t xw[4] = {xv[h].x, xv[h].y, xv[h].z, xv[h].w};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double c = n_tot * (double)((xw[i >> 2] >> (8 * (i & 3))) & 0xFFu) - s_S[16 * q + i];
            p = fma((i & 1) ? rv[h][i >> 1].y : rv[h][i >> 1].x, c, p);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0, 0);
#pragma unroll 1
    for (int q = 0; q < 8; q += 2) {
        fetch(1, q + 1);
        chain(0, q);
        fetch(0, min(q + 2, 7));
        chain(1, q + 1);
    }
    return p;
}

// What a block of projections shares: DESC descriptors' bits and the bits of
// the projections inside the margin, 176 in six words each.
template <int DESC>
struct ProjBlock {
    uint32_t bits[DESC][6], near[DESC][6];
    const uint8_t* x[DESC];
    uint32_t pre[DESC];  // inclusive prefix of the recomputes per descriptor
    double S[kDim];

    // The flagged projections of the block (their bits are 0 so far), one per
    // thread whichever descriptor and row they belong to; positive values set
    // their bit.  A flagged projection of 64 descriptors is one of about 15, so
    // a block's chains run side by side, beside other blocks' products.
    // Returns after a barrier.  counts: kCountSlots counters a line apart (one
    // address for every block's atomic would queue them).
    __device__ __forceinline__ void recompute(const double* __restrict__ R, double n_tot,
                                              unsigned long long* __restrict__ counts) {
        const int tid = threadIdx.x;
        if (tid < 64) {
            uint32_t carry = 0;
            for (int d0 = 0; d0 < DESC; d0 += 64) {
                uint32_t c = 0;
#pragma unroll
                for (int w = 0; w < 6; ++w) c += (uint32_t)__popc(near[d0 + tid][w]);
                const uint32_t incl = carry + wave_incl_scan(c, tid);
                pre[d0 + tid] = incl;
                carry = (uint32_t)__shfl((int)incl, 63);
            }
        }
        __syncthreads();
        const uint32_t total = pre[DESC - 1];
        for (uint32_t j = tid; j < total; j += 256) {
            // owner: the first descriptor whose prefix exceeds j
            uint32_t L = 0;
#pragma unroll
            for (uint32_t step = DESC / 2; step >= 1; step >>= 1)
                if (pre[L + step - 1] <= j) L += step;
            uint32_t kth = j - (L ? pre[L - 1] : 0u);
            int w = 0;
            uint32_t m = near[L][0];
            for (uint32_t c = (uint32_t)__popc(m); kth >= c; c = (uint32_t)__popc(m)) {
                kth -= c;
                m = near[L][++w];
            }
            for (uint32_t t = 0; t < kth; ++t) m &= m - 1;
            const int bit = __ffs(m) - 1;
            if (near_chain(x[L], R + (size_t)(32 * w + bit) * kDim, S, n_tot) > 0.0) atomicOr(&bits[L][w], 1u << bit);
        }
        if (tid == 0 && total) atomicAdd(counts + (blockIdx.x % kCountSlots) * kCountStride, (unsigned long long)total);
        __syncthreads();
    }
};

// Code and keys of one descriptor, from its 176 bits in six words.
__device__ __forceinline__ void store_code(const CodeOut& o, int row, const uint32_t* b) {
    gstore(reinterpret_cast<ulonglong2*>(o.codes) + row,
           make_ulonglong2((uint64_t)b[0] | ((uint64_t)b[1] << 32), (uint64_t)b[2] | ((uint64_t)b[3] << 32)));
    uint16_t* kp = reinterpret_cast<uint16_t*>(o.keys + 6 * (int64_t)row);
    gstore(kp, (uint16_t)b[4]);
    gstore(kp + 1, (uint16_t)(b[4] >> 16));
    gstore(kp + 2, (uint16_t)b[5]);
}

// BF16 hi+lo split on MFMA: D[16 rows][16 desc] = sum over 4 k-steps of
// (R_hi + R_lo)[rows][32 k] x X^T[32 k][desc] with v_mfma_f32_16x16x32_bf16.
// A block keeps all of R in registers, wavefront w the row tiles w, w + 4 and
// w + 8 of 11, and takes groups of tpg <= 4 tiles of 16 descriptors, n_groups
// in all, a grid apart: wavefront w widens tile w's descriptors (loaded during
// the group before) to bf16 fragments in LDS, every wavefront multiplies every
// tile by its rows, and wavefront k < 3 stores word k of codes and keys.
// (With R read from L2 for each group of 64 descriptors that was 1.1 GB at
// 800k descriptors.)  Where a tile's rows lie and go is worked out for
// kTileRun groups at once: the dependent loads behind it would not fit between
// two groups.
// Lane l holds descriptor l % 16 of a tile and rows 4 (l / 16) .. +3 of each
// row tile.  A value v is positive where its sign bit is clear, inside the
// margin M where that of M - |v| is (the difference of two fp32 numbers has
// the exact sign), so both tests are one shift each into a word of 12 bits.
// FUSED: a block takes one group, and recomputes what lies inside the margin
// itself; otherwise words with such bits go into the block's three segments
// of the near list (seg_cap entries each) for near_kernel.
// 800k descriptors: 89 us (123 with R from L2 for each wavefront and the bits
// unpacked in every lane), of which the products alone are 31 and the vector
// instructions around them 41; leaving out loads or stores changes nothing.
// 4000 descriptors: 10 us with the recompute (17.5 + 29 as four launches; three
// of its 256 registers are spilled, once per block).
template <bool FUSED>
__global__ __launch_bounds__(256, 2) void proj_mfma_kernel(const ImgDev* __restrict__ imgs,
                                                           const CodeOut* __restrict__ outs,
                                                           const RowChunk* __restrict__ tiles, int n_tiles, int tpg,
                                                           int n_groups, const uint4* __restrict__ frag,
                                                           const float* __restrict__ bias, float margin_coef,
                                                           const double* __restrict__ R,
                                                           const unsigned long long* __restrict__ S, double n_tot,
                                                           unsigned long long* __restrict__ counts,
                                                           NearEntry* __restrict__ near,
                                                           uint32_t* __restrict__ seg_count, uint32_t seg_cap) {
    constexpr int DESC = 16 * kProjTB;
    constexpr int kTileRun = FUSED ? 1 : 16;
    static_assert(kProjTB == 4, "a wavefront per tile");
    struct Tile {
        const uint8_t* x;
        uint64_t* codes;
        uint8_t* keys;
        int32_t img, row, nr, pad;
    };
    __shared__ __attribute__((aligned(16))) uint4 s_x[kProjTB][4][64];  // bf16 fragments [tile][k step][lane]
    __shared__ float s_margin[DESC];
    // [descriptor][4 wavefront + row group]: signs, margin hits << 16
    __shared__ __attribute__((aligned(16))) uint32_t s_out[DESC][20];
    __shared__ Tile s_tile[kTileRun][kProjTB];
    __shared__ ProjBlock<FUSED ? DESC : 1> blk;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = (int)uniform((uint32_t)tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const bool third = wv + 8 < kRowTiles;
    const int step = (int)gridDim.x;
    // tiles of the kTileRun groups from grp on (nr 0: none there)
    auto set_tiles = [&](int grp) {
        if (tid < kTileRun * kProjTB) {
            const int b = tid % kProjTB;
            const int gi = grp + (tid / kProjTB) * step;
            const int t = gi * tpg + b;
            Tile r{};
            if (gi < n_groups && b < tpg && t < n_tiles) {
                const RowChunk tc = tiles[t];
                const CodeOut o = outs[tc.img];
                r.x = imgs[tc.img].desc + (int64_t)tc.r0 * kDim;
                r.codes = o.codes + 2 * (int64_t)tc.r0;
                r.keys = o.keys + 6 * (int64_t)tc.r0;
                r.img = tc.img;
                r.row = tc.r0;
                r.nr = tc.nr;
            }
            s_tile[tid / kProjTB][b] = r;
        }
    };
    int grp = blockIdx.x;
    set_tiles(grp);
    if constexpr (FUSED)
        if (tid < kDim) blk.S[tid] = (double)S[tid];
    bf16x8 fr[3][4][2];
    float bv[3][4], mb[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int rt = k < 2 || third ? wv + 4 * k : wv;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            fr[k][ks][0] = load_frag(frag, ((0 * kRowTiles + rt) * 4 + ks) * 64 + lane);
            fr[k][ks][1] = load_frag(frag, ((1 * kRowTiles + rt) * 4 + ks) * 64 + lane);
        }
        const float4 bq = reinterpret_cast<const float4*>(bias)[rt * 4 + g];
        bv[k][0] = bq.x, bv[k][1] = bq.y, bv[k][2] = bq.z, bv[k][3] = bq.w;
#pragma unroll
        for (int i = 0; i < 4; ++i) mb[k][i] = 0x1p-20f * fabsf(bv[k][i]);
    }
    __syncthreads();
    // this lane's 8-byte pieces of its descriptor of this wavefront's tile of
    // group `slot` of the run
    uint2 w[4];
    bool live = false;
    auto fetch = [&](int slot) {
        const Tile& t = s_tile[slot][wv];
        live = n < t.nr;
        const uint8_t* x = t.x + n * kDim + 8 * g;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            w[ks] = live ? gload(reinterpret_cast<const uint2*>(x + 32 * ks)) : make_uint2(0u, 0u);
    };
    fetch(0);
    uint32_t cnt = 0;  // near-list entries so far (wavefronts 0 to 2)
    int slot = 0;
    for (; grp < n_groups; grp += step) {
        {
            uint32_t sq = 0;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                sq = __builtin_amdgcn_udot4(w[ks].x, w[ks].x, sq, false);
                sq = __builtin_amdgcn_udot4(w[ks].y, w[ks].y, sq, false);
                s_x[wv][ks][lane] = make_uint4(bf16_pair(w[ks].x, 0), bf16_pair(w[ks].x, 16), bf16_pair(w[ks].y, 0),
                                               bf16_pair(w[ks].y, 16));
            }
            sq += __shfl_xor(sq, 16);
            sq += __shfl_xor(sq, 32);
            if (g == 0) {
                // (rows past a tile's end are never inside the margin)
                s_margin[16 * wv + n] = live ? margin_coef * sqrtf((float)sq) + 0x1p-26f : -__builtin_inff();
                if constexpr (FUSED) blk.x[16 * wv + n] = s_tile[0][wv].x + (live ? n * kDim : 0);
            }
        }
        __syncthreads();
        const bool more = slot + 1 < kTileRun;
        if (more) fetch(slot + 1);
        // the fragments of a tile are read while the tile before it is multiplied
        struct Frags {
            bf16x8 x[4];
            float base;
        };
        auto frags = [&](int b) {
            Frags f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                union {
                    uint4 u;
                    bf16x8 v;
                } cv;
                cv.u = s_x[b][ks][lane];
                f.x[ks] = cv.v;
            }
            f.base = s_margin[16 * b + n];
            return f;
        };
        auto tile = [&](int b, auto nrt, const Frags& f) {
            constexpr int NRT = decltype(nrt)::value;
            f32x4 acc[NRT];
#pragma unroll
            for (int k = 0; k < NRT; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int k = 0; k < NRT; ++k)
                        acc[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[k][ks][h], f.x[ks], acc[k], 0, 0, 0);
            uint32_t neg = 0, far = 0;
#pragma unroll
            for (int k = NRT - 1; k >= 0; --k)
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    const float v = acc[k][i] - bv[k][i];
                    const float d = (f.base + mb[k][i]) - fabsf(v);
                    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(v), 31);
                    far = __builtin_amdgcn_alignbit(far, __float_as_uint(d), 31);
                }
            constexpr uint32_t kAll = (1u << (4 * NRT)) - 1u;
            s_out[16 * b + n][4 * wv + g] = (far & (neg ^ kAll)) | ((far ^ kAll) << 16);
        };
        auto product = [&](auto nrt) {
            Frags f[2];
            f[0] = frags(0);
            if constexpr (FUSED) {
                for (int b = 0; b < tpg; ++b) {
                    f[1] = frags(min(b + 1, tpg - 1));
                    __builtin_amdgcn_sched_barrier(0);
                    tile(b, nrt, f[0]);
                    f[0] = f[1];
                }
            } else {
#pragma unroll
                for (int b = 0; b < kProjTB; ++b) {
                    if (b + 1 < kProjTB) f[(b + 1) & 1] = frags(b + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    tile(b, nrt, f[b & 1]);
                }
            }
        };
        if (third)
            product(std::integral_constant<int, 3>{});
        else
            product(std::integral_constant<int, 2>{});
        __syncthreads();
        if (third) {
            // word wv of descriptor `lane` of the group: row tiles 4 wv .. + 3
            const Tile& t = s_tile[slot][g];
            const bool in = n < t.nr;
            uint32_t bits[2] = {0u, 0u}, nr[2] = {0u, 0u};
#pragma unroll
            for (int w4 = 0; w4 < 4; ++w4) {
                const uint4 q = *reinterpret_cast<const uint4*>(&s_out[lane][4 * w4]);
                const uint32_t v[4] = {q.x >> (4 * wv), q.y >> (4 * wv), q.z >> (4 * wv), q.w >> (4 * wv)};
#pragma unroll
                for (int gg = 0; gg < 4; ++gg) {
                    bits[w4 >> 1] |= (v[gg] & 0xFu) << (16 * (w4 & 1) + 4 * gg);
                    nr[w4 >> 1] |= ((v[gg] >> 16) & 0xFu) << (16 * (w4 & 1) + 4 * gg);
                }
            }
            if (!in) nr[0] = nr[1] = 0u;
            if constexpr (FUSED) {
                blk.bits[lane][2 * wv] = bits[0];
                blk.bits[lane][2 * wv + 1] = bits[1];
                blk.near[lane][2 * wv] = nr[0];
                blk.near[lane][2 * wv + 1] = nr[1];
            } else {
                if (in) {
                    if (wv < 2) {
                        gstore(t.codes + 2 * n + wv, (uint64_t)bits[0] | ((uint64_t)bits[1] << 32));
                    } else {
                        uint16_t* kp = reinterpret_cast<uint16_t*>(t.keys + 6 * n);
                        gstore(kp, (uint16_t)bits[0]);
                        gstore(kp + 1, (uint16_t)(bits[0] >> 16));
                        gstore(kp + 2, (uint16_t)bits[1]);
                    }
                }
                const bool flagged = (nr[0] | nr[1]) != 0;
                const uint64_t fm = __ballot(flagged);
                if (flagged)
                    gstore(reinterpret_cast<uint4*>(near + (size_t)(3 * blockIdx.x + wv) * seg_cap + cnt + mbcnt64(fm)),
                           make_uint4((uint32_t)t.img, (uint32_t)(t.row + n), nr[0], nr[1]));
                cnt += (uint32_t)__popcll(fm);
            }
        }
        if constexpr (FUSED) {
            __syncthreads();
            blk.recompute(R, n_tot, counts);
            if (tid < DESC) {
                const Tile& t = s_tile[0][tid >> 4];
                if (n < t.nr) store_code(CodeOut{t.codes, t.keys, 0}, n, blk.bits[tid]);
            }
        } else if (more) {
            ++slot;
        } else {
            __syncthreads();
            set_tiles(grp + step);
            __syncthreads();
            slot = 0;
            fetch(0);
        }
    }
    if constexpr (!FUSED)
        if (third && lane == 0) seg_count[3 * blockIdx.x + wv] = cnt;
}

// The recompute of the near list: a block takes word `word` of the near
// lists of kNearSegs projection blocks, a thread an entry and then a flagged
// projection.  Every lane needs another row of R, so half of the columns of R
// at a time are in LDS (16 bytes per lane from memory are a cache line per
// lane: 94.7 us at 800k descriptors and 190k projections), rows two doubles
// longer than that so that equal columns of different rows lie in all banks.
// 800k descriptors, 190k projections: 17.5 us (38 for a sort by row, a
// wavefront per 64 projections of one row, and a pass to store the results).
__global__ __launch_bounds__(kNearThreads) void near_kernel(const ImgDev* __restrict__ imgs,
                                                            const CodeOut* __restrict__ outs,
                                                            const NearEntry* __restrict__ near,
                                                            const uint32_t* __restrict__ seg_count, uint32_t seg_cap,
                                                            uint32_t n_lists, const double* __restrict__ R,
                                                            const unsigned long long* __restrict__ S, double n_tot,
                                                            unsigned long long* __restrict__ counts) {
    constexpr int kHalf = kDim / 2, kStride = kHalf + 2;
    constexpr int kWaves = kNearThreads / 64;
    __shared__ __attribute__((aligned(16))) double s_R[64 * kStride];  // 64 rows of one word
    __shared__ double s_S[kDim];
    __shared__ uint32_t s_pre[kNearThreads], s_wave[kWaves];
    __shared__ uint32_t s_mask[kNearThreads][2], s_bits[kNearThreads][2];
    __shared__ const uint8_t* s_xp[kNearThreads];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t word = blockIdx.x % 3, l0 = blockIdx.x / 3 * kNearSegs;
    const int rows = word < 2 ? 64 : kRows - 128;
    uint32_t n_seg[kNearSegs], n = 0;
#pragma unroll
    for (int i = 0; i < kNearSegs; ++i) {
        n_seg[i] = l0 + i < n_lists ? uniform(seg_count[3 * (l0 + i) + word]) : 0u;
        n += n_seg[i];
    }
    if (n == 0) return;
    if (tid < kDim) s_S[tid] = (double)S[tid];
    uint32_t n_jobs = 0;
    for (uint32_t e0 = 0; e0 < n; e0 += kNearThreads) {
        uint32_t at = e0 + tid, li = 0;
        const bool has = at < n;
#pragma unroll
        for (int i = 0; i + 1 < kNearSegs; ++i)
            if (li == (uint32_t)i && at >= n_seg[i]) at -= n_seg[i], ++li;
        uint4 e = make_uint4(0u, 0u, 0u, 0u);
        if (has) e = gload(reinterpret_cast<const uint4*>(near + (size_t)(3 * (l0 + li) + word) * seg_cap + at));
        s_xp[tid] = imgs[e.x].desc + (int64_t)(int32_t)e.y * kDim;
        s_mask[tid][0] = e.z;
        s_mask[tid][1] = e.w;
        s_bits[tid][0] = s_bits[tid][1] = 0u;
        uint32_t incl = wave_incl_scan((uint32_t)(__popc(e.z) + __popc(e.w)), lane);
        if (lane == 63) s_wave[wv] = incl;
        __syncthreads();
        uint32_t total = 0;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
            if (i == wv) incl += total;
            total += s_wave[i];
        }
        s_pre[tid] = incl;
        n_jobs += total;
        for (uint32_t j0 = 0; j0 < total; j0 += kNearThreads) {
            __syncthreads();  // s_pre is there; the other half of R is read
            const uint32_t j = j0 + tid;
            const bool act = j < total;
            // owner: the first entry whose prefix exceeds j; its kth set bit
            uint32_t L = 0;
#pragma unroll
            for (uint32_t st = kNearThreads / 2; st >= 1; st >>= 1)
                if (act && s_pre[L + st - 1] <= j) L += st;
            uint32_t kth = act ? j - (L ? s_pre[L - 1] : 0u) : 0u;
            uint32_t m = s_mask[L][0];
            const uint32_t c0 = (uint32_t)__popc(m);
            const bool up = kth >= c0;
            if (up) {
                kth -= c0;
                m = s_mask[L][1];
            }
            for (uint32_t t = 0; t < kth; ++t) m &= m - 1;
            const int bit = act ? __ffs(m) - 1 : 0;
            const uint4* xp = reinterpret_cast<const uint4*>(s_xp[L]);
            const double* rp = s_R + (act ? (up ? 32 : 0) + bit : 0) * kStride;
            double p = 0.0;
            for (int half = 0; half < 2; ++half) {
                if (half) __syncthreads();
                for (int i = tid; i < rows * (kHalf / 2); i += kNearThreads) {
                    const int r = i / (kHalf / 2), c = i % (kHalf / 2);
                    *reinterpret_cast<double2*>(s_R + r * kStride + 2 * c) =
                        *reinterpret_cast<const double2*>(R + (size_t)(64 * word + r) * kDim + half * kHalf + 2 * c);
                }
                uint4 xv[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) xv[q] = gload(xp + 4 * half + q);
                __syncthreads();
                if (act) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t xw[4] = {xv[q].x, xv[q].y, xv[q].z, xv[q].w};
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const double c = n_tot * (double)((xw[i >> 2] >> (8 * (i & 3))) & 0xFFu) -
                                             s_S[half * kHalf + 16 * q + i];
                            p = fma(rp[16 * q + i], c, p);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            if (act && p > 0.0) atomicOr(&s_bits[L][up ? 1 : 0], 1u << bit);
        }
        __syncthreads();
        const uint32_t b0 = s_bits[tid][0], b1 = s_bits[tid][1];
        if (has && (b0 | b1)) {
            const CodeOut o = outs[e.x];
            const int64_t row = (int32_t)e.y;
            if (word < 2) {
                o.codes[2 * row + word] |= (uint64_t)b0 | ((uint64_t)b1 << 32);
            } else {
                uint16_t* kp = reinterpret_cast<uint16_t*>(o.keys + 6 * row);
                kp[0] |= (uint16_t)b0;
                kp[1] |= (uint16_t)(b0 >> 16);
                kp[2] |= (uint16_t)b1;
            }
        }
        __syncthreads();
    }
    if (tid == 0) atomicAdd(counts + (blockIdx.x % kCountSlots) * kCountStride, (unsigned long long)n_jobs);
}

// Plain FP32 form: one thread per descriptor, 176 fp32 FMA chains over the
// descriptor held in registers; the rows are wave-uniform scalar loads.  What
// lies inside the margin goes into the block's three segments of the near list
// (256 entries each), in any order.
// Bound by the fp32 multiply-adds: 240k descriptors 330 us, and 19 for near_kernel
// (506 us with the recompute in this kernel).
__global__ __launch_bounds__(256) void proj_fp32_kernel(const ImgDev* __restrict__ imgs,
                                                        const CodeOut* __restrict__ outs,
                                                        const RowChunk* __restrict__ tiles, int n_tiles,
                                                        const float* __restrict__ R32,
                                                        const float* __restrict__ bias, float margin_coef,
                                                        NearEntry* __restrict__ near,
                                                        uint32_t* __restrict__ seg_count) {
    __shared__ uint32_t s_cnt[3];
    const int tid = threadIdx.x;
    if (tid < 3) s_cnt[tid] = 0u;
    __syncthreads();
    const int t = blockIdx.x * blockDim.x + tid;
    const int tile = min(t >> 4, n_tiles - 1), n = t & 15;
    const RowChunk tc = tiles[tile];
    const bool live = (t >> 4) < n_tiles && n < tc.nr;
    const uint4* xp = reinterpret_cast<const uint4*>(imgs[tc.img].desc + (int64_t)(tc.r0 + (live ? n : 0)) * kDim);
    float xf[kDim];
    uint32_t sq = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const uint4 w = xp[c];
        const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            sq = __builtin_amdgcn_udot4(ws[a], ws[a], sq, false);
#pragma unroll
            for (int b = 0; b < 4; ++b) xf[c * 16 + a * 4 + b] = (float)((ws[a] >> (8 * b)) & 0xFFu);
        }
    }
    const float base_margin = margin_coef * sqrtf((float)sq) + 0x1p-26f;
    uint64_t w[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        uint64_t m = 0;
        const int rows = k < 2 ? 64 : kRows - 128;
        for (int rr = 0; rr < rows; ++rr) {
            const int r = 64 * k + rr;
            const float* rp = R32 + r * kDim;
            float acc = 0.f;
#pragma unroll
            for (int i = 0; i < kDim; ++i) acc = fmaf(rp[i], xf[i], acc);
            const float bv = bias[r];
            const float v = acc - bv;
            const float M = base_margin + 0x1p-20f * fabsf(bv);
            const bool nr = !(fabsf(v) > M);
            const bool bit = !nr && v > 0.f;
            w[k] |= (uint64_t)bit << rr;
            m |= (uint64_t)nr << rr;
        }
        if (live && m != 0)
            gstore(reinterpret_cast<uint4*>(near + (size_t)(3 * blockIdx.x + k) * 256 + atomicAdd(&s_cnt[k], 1u)),
                   make_uint4((uint32_t)tc.img, (uint32_t)(tc.r0 + n), (uint32_t)m, (uint32_t)(m >> 32)));
    }
    if (live) {
        const uint32_t b[6] = {(uint32_t)w[0], (uint32_t)(w[0] >> 32), (uint32_t)w[1], (uint32_t)(w[1] >> 32),
                               (uint32_t)w[2], (uint32_t)(w[2] >> 32)};
        store_code(outs[tc.img], tc.r0 + n, b);
    }
    __syncthreads();
    if (tid < 3) seg_count[3 * blockIdx.x + tid] = s_cnt[tid];
}

// ------------------------------------------------------------------ bucket tables
// One block of kBucketWaves wavefronts per (train image, table): a stable
// counting sort of the 8-bit keys into 256 buckets (ascending index inside a
// bucket).  Wave w owns a contiguous slice of the entries: it counts its
// slice's keys, the block scans the bucket totals and gives each wave its
// start inside every bucket, then each wave scatters its slice in order.
// Ranks inside a 64-wide chunk come from eight key-bit ballots.

// Keys and index of an entry of table t, for the matcher's union test (a
// candidate counts in the first table whose key it shares with the query).
// Low word: the keys of tables 0-3 before t, 0 in the other bytes.  High word:
// the index above 16 bits that hold key 4 in table 5's entries and else 0x100,
// which no key equals.
__device__ __forceinline__ uint64_t entry_word(int t, uint32_t k03, uint32_t k45, uint32_t j) {
    const uint32_t lo = t >= 4 ? k03 : k03 & ~(~0u << (8 * t));
    const uint32_t hi = (j << 16) | (t == 5 ? k45 & 0xFFu : 0x100u);
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

template <bool EPI>
__global__ __launch_bounds__(64 * kBucketWaves) void bucket_kernel(const ImgDev* __restrict__ imgs,
                                                                   const TableOut* __restrict__ touts,
                                                                   const int32_t* __restrict__ train_list,
                                                                   int32_t n_train, ItemArgs ia) {
    // blocks after the tables' make the work items
    if ((int)blockIdx.x >= n_train * kTables) {
        make_item(ia, imgs, ((int32_t)blockIdx.x - n_train * kTables) * (64 * kBucketWaves) + (int32_t)threadIdx.x);
        return;
    }
    __shared__ uint32_t cnt[kBucketWaves][256];  // per-wave counts, then per-wave write positions
    __shared__ uint32_t wsum[4];
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int m = train_list[blockIdx.x / kTables];
    const int t = blockIdx.x % kTables;
    const ImgDev im = imgs[m];
    const TableOut to = touts[m];
    const int n = im.n;
    // this wave's slice [lo, hi), a whole number of 64-entry chunks
    const int per = ((n + 64 * kBucketWaves - 1) / (64 * kBucketWaves)) * 64;
    const int lo = min(n, wv * per), hi = min(n, lo + per);
#pragma unroll
    for (int i = 0; i < 4; ++i) cnt[wv][4 * lane + i] = 0;
    __syncthreads();
#pragma unroll 4
    for (int j = lo + lane; j < hi; j += 64) atomicAdd(&cnt[wv][gload(im.keys + 6 * (int64_t)j + t)], 1u);
    __syncthreads();
    // thread b < 256 of the block owns bucket b
    static_assert(64 * kBucketWaves >= 256, "a thread per bucket");
    const int bk = threadIdx.x;
    uint32_t c[kBucketWaves], tot = 0, incl = 0;
    if (bk < 256) {
#pragma unroll
        for (int w = 0; w < kBucketWaves; ++w) {
            c[w] = cnt[w][bk];
            tot += c[w];
        }
        incl = wave_incl_scan(tot, lane);
        if (lane == 63) wsum[wv] = incl;
    }
    __syncthreads();
    if (bk < 256) {
        uint32_t start = incl - tot;
        for (int w = 0; w < wv; ++w) start += wsum[w];
        uint32_t* off = to.off + t * kOffStride;
        gstore(off + bk, start);
        if (bk == 255) gstore(off + 256, start + tot);
#pragma unroll
        for (int w = 0; w < kBucketWaves; ++w) {
            cnt[w][bk] = start;
            start += c[w];
        }
    }
    __syncthreads();
    ulonglong2* out_code = reinterpret_cast<ulonglong2*>(to.ent) + (int64_t)t * n;
    uint64_t* out_kid = reinterpret_cast<uint64_t*>(to.ent + (size_t)kTables * n * 16) + (int64_t)t * n;
    float2* out_kp = reinterpret_cast<float2*>(to.ent + (size_t)kTables * n * 24) + (int64_t)t * n;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t* wc = cnt[wv];
    for (int c0 = lo; c0 < hi; c0 += 64) {
        const int j = c0 + lane;
        const bool valid = j < hi;
        const uint32_t key = valid ? gload(im.keys + 6 * (int64_t)j + t) : 0u;
        uint64_t eq = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool kb = (key >> b) & 1u;
            const uint64_t bm = __ballot(kb);
            eq &= kb ? bm : ~bm;
        }
        const uint32_t rank = __popcll(eq & lt_mask);
        uint32_t pos = 0;
        if (valid) pos = wc[key] + rank;
        wave_sync();  // every lane has read its bucket's position before the first lane advances it
        if (valid) {
            const uint16_t* kp = reinterpret_cast<const uint16_t*>(im.keys + 6 * (int64_t)j);
            gstore(out_code + pos, gload(reinterpret_cast<const ulonglong2*>(im.codes) + j));
            const uint32_t k03 = (uint32_t)gload(kp) | ((uint32_t)gload(kp + 1) << 16);
            gstore(out_kid + pos, entry_word(t, k03, gload(kp + 2), (uint32_t)j));
            if constexpr (EPI) gstore(out_kp + pos, gload(reinterpret_cast<const float2*>(im.kp) + j));
            if (rank == 0) wc[key] = pos + (uint32_t)__popcll(eq);
        }
        wave_sync();
    }
}

// ------------------------------------------------------------------ launchers
hipError_t launch_fill_u64(hipStream_t s, unsigned long long* p, int64_t n, unsigned long long v) {
    if (n <= 0) return hipSuccess;
    CH_LAUNCH(fill_u64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipSuccess;
}

hipError_t launch_fill_u32(hipStream_t s, uint32_t* p, int64_t n, uint32_t v) {
    if (n <= 0) return hipSuccess;
    CH_LAUNCH(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipSuccess;
}

hipError_t launch_make_items(hipStream_t s, const ItemArgs& a, const ImgDev* imgs) {
    const unsigned threads = (unsigned)std::max(a.n_items, kCtlWords);
    CH_LAUNCH(make_items_kernel, dim3((threads + 255) / 256), dim3(256), 0, s, a, imgs);
    return hipSuccess;
}

hipError_t launch_colsum(hipStream_t s, const ImgDev* imgs, const RowChunk* chunks, int n_chunks,
                         unsigned long long* S) {
    if (n_chunks <= 0) return hipSuccess;
    CH_LAUNCH(colsum_kernel<false>, dim3(n_chunks), dim3(256), 0, s, imgs, chunks, S, (const double*)nullptr, 0.0,
              (float*)nullptr, (unsigned long long*)nullptr, (unsigned long long*)nullptr);
    return hipSuccess;
}

hipError_t launch_colsum_bias(hipStream_t s, const ImgDev* imgs, const RowChunk* chunks, int n_chunks,
                              unsigned long long* S, const double* Rt, double n_tot, float* bias,
                              unsigned long long* next_S, unsigned long long* counts) {
    if (n_chunks <= 0) return hipSuccess;
    CH_LAUNCH(colsum_kernel<true>, dim3(n_chunks), dim3(256), 0, s, imgs, chunks, S, Rt, n_tot, bias, next_S, counts);
    return hipSuccess;
}

hipError_t launch_bias(hipStream_t s, const double* Rt, const unsigned long long* S, double n_tot, float* bias) {
    CH_LAUNCH(bias_kernel, dim3(1), dim3(256), 0, s, Rt, S, n_tot, bias);
    return hipSuccess;
}

// The recompute of what a projection of plan pl left in its near list.
static hipError_t launch_near(hipStream_t s, const ImgDev* imgs, const CodeOut* outs, const ProjPlan& pl,
                              const NearEntry* list, const uint32_t* seg_count, const double* R,
                              const unsigned long long* S, double n_tot, unsigned long long* counts) {
    CH_LAUNCH(near_kernel, dim3((unsigned)((pl.grid + kNearSegs - 1) / kNearSegs * 3)), dim3(kNearThreads), 0, s, imgs,
              outs, list, seg_count, pl.seg_cap(), (uint32_t)pl.grid, R, S, n_tot, counts);
    return hipSuccess;
}

hipError_t launch_proj_mfma(hipStream_t s, const ImgDev* imgs, const CodeOut* outs, const RowChunk* tiles, int n_tiles,
                            const uint4* frag, const float* bias, float margin, const double* R,
                            const unsigned long long* S, double n_tot, unsigned long long* counts, const ProjPlan& pl,
                            void* near) {
    if (n_tiles <= 0) return hipSuccess;
    if (pl.fused) {
        CH_LAUNCH(proj_mfma_kernel<true>, dim3((unsigned)pl.grid), dim3(256), 0, s, imgs, outs, tiles, n_tiles, pl.tpg,
                  pl.groups, frag, bias, margin, R, S, n_tot, counts, (NearEntry*)nullptr, (uint32_t*)nullptr, 0u);
        return hipSuccess;
    }
    uint32_t* seg_count = static_cast<uint32_t*>(near);
    NearEntry* list = reinterpret_cast<NearEntry*>(static_cast<uint8_t*>(near) + pl.count_bytes());
    CH_LAUNCH(proj_mfma_kernel<false>, dim3((unsigned)pl.grid), dim3(256), 0, s, imgs, outs, tiles, n_tiles, pl.tpg,
              pl.groups, frag, bias, margin, R, S, n_tot, counts, list, seg_count, pl.seg_cap());
    return launch_near(s, imgs, outs, pl, list, seg_count, R, S, n_tot, counts);
}

hipError_t launch_proj_fp32(hipStream_t s, const ImgDev* imgs, const CodeOut* outs, const RowChunk* tiles, int n_tiles,
                            const float* R32, const float* bias, float margin, const double* R,
                            const unsigned long long* S, double n_tot, unsigned long long* counts, const ProjPlan& pl,
                            void* near) {
    if (n_tiles <= 0) return hipSuccess;
    uint32_t* seg_count = static_cast<uint32_t*>(near);
    NearEntry* list = reinterpret_cast<NearEntry*>(static_cast<uint8_t*>(near) + pl.count_bytes());
    CH_LAUNCH(proj_fp32_kernel, dim3((unsigned)pl.grid), dim3(256), 0, s, imgs, outs, tiles, n_tiles, R32, bias, margin,
              list, seg_count);
    return launch_near(s, imgs, outs, pl, list, seg_count, R, S, n_tot, counts);
}

hipError_t launch_bucket(hipStream_t s, bool epi, const ImgDev* imgs, const TableOut* touts, const int32_t* train_list,
                         int n_train, const ItemArgs* items) {
    const ItemArgs ia = items ? *items : ItemArgs{};
    const unsigned per = 64 * kBucketWaves;
    const unsigned grid = (unsigned)n_train * kTables +
                          (items ? ((unsigned)std::max(ia.n_items, kCtlWords) + per - 1) / per : 0u);
    if (grid == 0) return hipSuccess;
    if (epi)
        CH_LAUNCH(bucket_kernel<true>, dim3(grid), dim3(per), 0, s, imgs, touts, train_list, n_train, ia);
    else
        CH_LAUNCH(bucket_kernel<false>, dim3(grid), dim3(per), 0, s, imgs, touts, train_list, n_train, ia);
    return hipSuccess;
}

}  // namespace cashash
