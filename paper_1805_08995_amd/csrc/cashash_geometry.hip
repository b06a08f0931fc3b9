// Geometry-aware first stage on gfx950 (Sec. 3.1 of the paper): the
// largest-scale fifth of each image's features is matched first, a
// fundamental matrix is estimated from each pair's matches, and only pairs
// whose matches are mostly inliers of it go on to epipolar-guided matching
// (Eq. 1-2).  The paper does not spell out its estimator; this one is RANSAC
// over Hartley-normalised eight-point hypotheses with a least-squares refit:
//
//   subset      ceil(n num / den) largest scales (IEEE total order of the
//               float32 value), lower index first on ties, ascending order
//   sampling    Floyd's algorithm over the pair's match list, one 32-bit
//               uniform draw per pick: v = floor(r (j + 1) / 2^32) for
//               j = n-8 .. n-1, replaced by j if already taken
//   hypothesis  null vector (f8 = 1) of the 8 x 9 design matrix of the
//               normalised sample by Gaussian elimination with partial
//               pivoting; rank 2 by F <- F (I - v v^T), v the eigenvector of
//               F^T F with the smallest eigenvalue (cyclic Jacobi, 6 sweeps);
//               back to pixels with F <- T_t^T F T_q
//   inlier      e^2 <= thr^2 (a^2 + b^2) with (a, b, c) = F (x, y, 1) and
//               e = a x' + b y' + c (the band test of Eq. 2)
//   best        most inliers, lowest hypothesis index on ties
//   refit       smallest eigenvector of A^T A over the best's inliers (cyclic
//               Jacobi, 10 sweeps), rank 2, pixels; inliers counted again
//   accept      n >= min_matches and 3 inliers >= 2 n
//
// Every step is binary64 in the order written (the library is compiled
// without fp contraction), and every sum runs sequentially in match order, so
// results are reproducible bit for bit.  Jacobi rotations use the symmetric
// Schur pair theta = (a_qq - a_pp) / (2 a_pq), t = sign(theta) / (|theta| +
// sqrt(theta^2 + 1)), c = 1 / sqrt(t^2 + 1), s = t c, applied to columns p, q,
// then rows p, q, then to the accumulated eigenvectors; planes with a_pq == 0
// are skipped.
#include "cashash_device.h"
#include "cashash_launch.h"

namespace cashash {

namespace {

constexpr double kSqrt2 = 1.4142135623730951;
enum { kAccept = 0, kFewMatches = 1, kDegenerate = 2, kFewInliers = 3 };

// IEEE total order of a float32 as an unsigned key (larger key, larger value).
__device__ __forceinline__ uint32_t scale_key(float s) {
    const uint32_t b = __float_as_uint(s);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Exclusive rank of `flag` among the block's 256 threads, in thread order,
// and the block's total.  wtot: 4 words of LDS.  Contains two barriers.
__device__ __forceinline__ uint32_t block_rank(bool flag, uint32_t* wtot, uint32_t* total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned long long b = __ballot(flag);
    if (lane == 0) wtot[wv] = (uint32_t)__popcll(b);
    __syncthreads();
    uint32_t r = (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
    for (int w = 0; w < wv; ++w) r += wtot[w];
    *total = wtot[0] + wtot[1] + wtot[2] + wtot[3];
    __syncthreads();
    return r;
}

}  // namespace

// ---------------------------------------------------------------- top scale
// One block per image.  Radix select over the 32-bit order keys, eight bits
// per pass from the top: each pass histograms the keys that share the digits
// chosen so far and picks the bin holding the rem-th largest.  The threshold
// key T and the number rem of keys equal to T that are taken come out of the
// fourth pass; a final pass writes, in index order, every key above T and the
// first rem keys equal to T.
__global__ __launch_bounds__(256) void top_scale_kernel(const SelectImg* __restrict__ imgs) {
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_pick[2];
    __shared__ uint32_t wtot[4];
    const SelectImg im = imgs[blockIdx.x];
    if (im.m <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63;
    uint32_t prefix = 0, pmask = 0, rem = (uint32_t)im.m;
    for (int shift = 24; shift >= 0; shift -= 8) {
        hist[tid] = 0;
        __syncthreads();
        for (int i = tid; i < im.n; i += 256) {
            const uint32_t k = scale_key(im.scale[i]);
            if ((k & pmask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (tid < 64) {
            // lane l holds bins 255-4l .. 252-4l, descending
            const int b0 = 255 - 4 * lane;
            const uint32_t h0 = hist[b0], h1 = hist[b0 - 1], h2 = hist[b0 - 2], h3 = hist[b0 - 3];
            const uint32_t sum = h0 + h1 + h2 + h3;
            uint32_t inc = sum;
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t v = __shfl_up(inc, d);
                if (lane >= d) inc += v;
            }
            const unsigned long long hit = __ballot(inc >= rem);
            if (lane == __ffsll((long long)hit) - 1) {
                uint32_t acc = inc - sum;
                int b = b0;
                if (acc + h0 < rem) {
                    acc += h0;
                    b = b0 - 1;
                    if (acc + h1 < rem) {
                        acc += h1;
                        b = b0 - 2;
                        if (acc + h2 < rem) {
                            acc += h2;
                            b = b0 - 3;
                        }
                    }
                }
                s_pick[0] = (uint32_t)b;
                s_pick[1] = rem - acc;
            }
        }
        __syncthreads();
        prefix |= s_pick[0] << shift;
        pmask |= 255u << shift;
        rem = s_pick[1];
    }
    uint32_t base = 0, base_eq = 0;
    for (int c0 = 0; c0 < im.n; c0 += 256) {
        const int i = c0 + tid;
        const uint32_t k = i < im.n ? scale_key(im.scale[i]) : 0u;
        const bool eq = i < im.n && k == prefix;
        uint32_t n_eq, n_take;
        const uint32_t eq_rank = base_eq + block_rank(eq, wtot, &n_eq);
        const bool take = (i < im.n && k > prefix) || (eq && eq_rank < rem);
        const uint32_t pos = base + block_rank(take, wtot, &n_take);
        if (take && pos < (uint32_t)im.m) im.rows_out[pos] = i;
        base += n_take;
        base_eq += n_eq;
    }
}

// ---------------------------------------------------------------- row gather
// 8 threads per row: each copies 16 descriptor bytes; threads 0-2 of the row
// also copy the code, the keys and the keypoint.  Rows outside the source
// image set bit 0 of *err and are skipped.
__global__ __launch_bounds__(256) void gather_rows_kernel(const GatherImg* __restrict__ imgs,
                                                          const RowChunk* __restrict__ chunks, int n_chunks,
                                                          unsigned* __restrict__ err) {
    const int rr = threadIdx.x >> 3, part = threadIdx.x & 7;
    for (int c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const RowChunk ch = chunks[c];
        if (rr >= ch.nr) continue;
        const GatherImg g = imgs[ch.img];
        const int j = ch.r0 + rr;
        const int32_t src = g.rows[j];
        if (src < 0 || src >= g.n) {
            if (part == 0) atomicOr(err, 1u);
            continue;
        }
        if (g.o_desc)
            reinterpret_cast<uint4*>(g.o_desc + (size_t)j * kDim)[part] =
                reinterpret_cast<const uint4*>(g.desc + (size_t)src * kDim)[part];
        if (part == 0 && g.o_codes) {
            g.o_codes[2 * (size_t)j] = g.codes[2 * (size_t)src];
            g.o_codes[2 * (size_t)j + 1] = g.codes[2 * (size_t)src + 1];
        }
        if (part == 1 && g.o_keys) {
            const uint16_t* s = reinterpret_cast<const uint16_t*>(g.keys + (size_t)src * kTables);
            uint16_t* d = reinterpret_cast<uint16_t*>(g.o_keys + (size_t)j * kTables);
            d[0] = s[0];
            d[1] = s[1];
            d[2] = s[2];
        }
        if (part == 2 && g.o_kp) {
            g.o_kp[2 * (size_t)j] = g.kp[2 * (size_t)src];
            g.o_kp[2 * (size_t)j + 1] = g.kp[2 * (size_t)src + 1];
        }
    }
}

// ---------------------------------------------------------------- fundamental matrix
namespace {

struct Norm2 {
    double s, cx, cy;
};

// Normalised coordinates of a pixel point.
__device__ __forceinline__ double nx(const Norm2& N, float x) { return N.s * ((double)x - N.cx); }
__device__ __forceinline__ double ny(const Norm2& N, float y) { return N.s * ((double)y - N.cy); }

// Eq. 2 band test with d^2 = dd.
__device__ __forceinline__ bool inlier(const double (&F)[9], float4 m, double dd) {
    const double x = (double)m.x, y = (double)m.y;
    const double la = (F[0] * x + F[1] * y) + F[2];
    const double lb = (F[3] * x + F[4] * y) + F[5];
    const double lc = (F[6] * x + F[7] * y) + F[8];
    const double e = (la * (double)m.z + lb * (double)m.w) + lc;
    return e * e <= dd * (la * la + lb * lb);
}

// One symmetric Schur rotation's (c, s) for plane (p, q).
__device__ __forceinline__ void schur(double app, double aqq, double apq, double& c, double& s) {
    const double theta = (aqq - app) / (2.0 * apq);
    double t = 1.0 / (fabs(theta) + sqrt(theta * theta + 1.0));
    if (theta < 0.0) t = -t;
    c = 1.0 / sqrt(t * t + 1.0);
    s = t * c;
}

// F <- F (I - v v^T) with v the eigenvector of F^T F of the smallest
// eigenvalue; 3 x 3 cyclic Jacobi held in registers.
__device__ __forceinline__ void rank2(double (&F)[9]) {
    double M[3][3], V[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            M[i][j] = (F[i] * F[j] + F[3 + i] * F[3 + j]) + F[6 + i] * F[6 + j];
            V[i][j] = i == j ? 1.0 : 0.0;
        }
#pragma unroll 1
    for (int sw = 0; sw < kJacobiSweeps3; ++sw) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = p + 1; q < 3; ++q) {
                if (M[p][q] == 0.0) continue;
                double c, s;
                schur(M[p][p], M[q][q], M[p][q], c, s);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double akp = M[k][p], akq = M[k][q];
                    M[k][p] = c * akp - s * akq;
                    M[k][q] = s * akp + c * akq;
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double apk = M[p][k], aqk = M[q][k];
                    M[p][k] = c * apk - s * aqk;
                    M[q][k] = s * apk + c * aqk;
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double vkp = V[k][p], vkq = V[k][q];
                    V[k][p] = c * vkp - s * vkq;
                    V[k][q] = s * vkp + c * vkq;
                }
            }
    }
    // smallest diagonal entry, first on ties.  The entries pass through an
    // empty asm so the selects below stay register selects (otherwise the
    // compiler turns them into one indexed load and keeps M, V in scratch).
    double d0 = M[0][0], d1 = M[1][1], d2 = M[2][2];
    double w00 = V[0][0], w10 = V[1][0], w20 = V[2][0], w01 = V[0][1], w11 = V[1][1], w21 = V[2][1];
    double w02 = V[0][2], w12 = V[1][2], w22 = V[2][2];
    asm volatile("" : "+v"(d0), "+v"(d1), "+v"(d2), "+v"(w00), "+v"(w10), "+v"(w20));
    asm volatile("" : "+v"(w01), "+v"(w11), "+v"(w21), "+v"(w02), "+v"(w12), "+v"(w22));
    double dmin = d0, v0 = w00, v1 = w10, v2 = w20;
    if (d1 < dmin) {
        dmin = d1;
        v0 = w01;
        v1 = w11;
        v2 = w21;
    }
    if (d2 < dmin) {
        v0 = w02;
        v1 = w12;
        v2 = w22;
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double w = (F[3 * i] * v0 + F[3 * i + 1] * v1) + F[3 * i + 2] * v2;
        F[3 * i + 0] = F[3 * i + 0] - w * v0;
        F[3 * i + 1] = F[3 * i + 1] - w * v1;
        F[3 * i + 2] = F[3 * i + 2] - w * v2;
    }
}

// Normalised-coordinate matrix back to pixels: F = T_t^T Fn T_q with
// T = [[s, 0, -s cx], [0, s, -s cy], [0, 0, 1]].
__device__ __forceinline__ void to_pixels(const double (&Fn)[9], const Norm2& Q, const Norm2& T, double (&F)[9]) {
    const double txq = -(Q.s * Q.cx), tyq = -(Q.s * Q.cy);
    const double txt = -(T.s * T.cx), tyt = -(T.s * T.cy);
    double G[9];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        G[3 * i + 0] = Fn[3 * i + 0] * Q.s;
        G[3 * i + 1] = Fn[3 * i + 1] * Q.s;
        G[3 * i + 2] = (Fn[3 * i + 0] * txq + Fn[3 * i + 1] * tyq) + Fn[3 * i + 2];
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        F[j] = T.s * G[j];
        F[3 + j] = T.s * G[3 + j];
        F[6 + j] = (txt * G[j] + tyt * G[3 + j]) + G[6 + j];
    }
}

// Design row of p'^T F p = 0 for normalised (x, y) <-> (u, v), F row-major.
__device__ __forceinline__ void design_row(double x, double y, double u, double v, double* a) {
    a[0] = u * x;
    a[1] = u * y;
    a[2] = u;
    a[3] = v * x;
    a[4] = v * y;
    a[5] = v;
    a[6] = x;
    a[7] = y;
    a[8] = 1.0;
}

// Null vector of the 8 x 9 matrix with f8 = 1 (partial pivoting, first row
// of the largest |a| on ties); false if a pivot is exactly zero.
__device__ __forceinline__ bool null8(double (&A)[8][9], double (&f)[9]) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        double best = fabs(A[c][c]);
        int p = c;
#pragma unroll
        for (int r = c + 1; r < 8; ++r) {
            const double v = fabs(A[r][c]);
            if (v > best) {
                best = v;
                p = r;
            }
        }
        if (best == 0.0) return false;
#pragma unroll
        for (int r = c + 1; r < 8; ++r)
            if (p == r) {
#pragma unroll
                for (int k = c; k < 9; ++k) {
                    const double t = A[c][k];
                    A[c][k] = A[r][k];
                    A[r][k] = t;
                }
            }
#pragma unroll
        for (int r = c + 1; r < 8; ++r) {
            const double g = A[r][c] / A[c][c];
#pragma unroll
            for (int k = c + 1; k < 9; ++k) A[r][k] = A[r][k] - g * A[c][k];
        }
    }
    f[8] = 1.0;
#pragma unroll
    for (int c = 7; c >= 0; --c) {
        double acc = 0.0;
#pragma unroll
        for (int k = c + 1; k < 9; ++k) acc = acc + A[c][k] * f[k];
        f[c] = -(acc / A[c][c]);
    }
    return true;
}

}  // namespace

// The estimator runs as three kernels: the fit of the best hypothesis up to the
// refit's normal matrix (a block per pair), the refit's eigenvector (27 lanes per
// pair) and the inlier count of its matrix (a block per pair).  The 360 rotations
// of the 9 x 9 Jacobi are one long chain of dependent divisions and square roots;
// in one kernel they kept a 256-thread block of 253 registers waiting, two blocks
// per CU, and everything sequential in match order ran in one thread: 667 us for
// 600 pairs of 400 matches (256 hypotheses each), now 161 + 154 + 4 us.  What is
// left is the binary64 work of the hypotheses (19 thousand VALU instructions per
// wavefront of the fit; four tests at a time or a third block per CU with its
// spills changed nothing) and the rotations' chain.
// The fit's design rows take 18 KB of LDS, so above about 3950 points per query
// image one block fits a CU (the one kernel had two up to 4800): 600 pairs of 400
// matches on images of 3800 / 4400 points 382 / 440 us per call, against 698 / 722.

// Sequential sum of v over the first n lanes of consecutive 64-lane chunks,
// s = ((s + v_0) + v_1) + .. : the lanes hold a chunk's values, the sum is
// uniform.
__device__ __forceinline__ double add_lanes(double s, double v, int n) {
    auto lane_value = [&](int i) {
        const uint64_t u = (uint64_t)__double_as_longlong(v);
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, i), hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), i);
        return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
    };
    if (n == 64) {
#pragma unroll
        for (int i = 0; i < 64; ++i) s = s + lane_value(i);
    } else {
        for (int i = 0; i < n; ++i) s = s + lane_value(i);
    }
    return s;
}

// One block of 256 threads per pair.  The pair's stage-1 matches are
// compacted (ascending query order) into LDS as (x, y, x', y'); the four waves
// take one coordinate's sum each, then two the distance sums (values by lane,
// sums in match order); each thread runs hypotheses h = tid, tid + 256, ...
// entirely in registers and counts their inliers against the LDS list; the
// block picks the best; its inliers' design rows are laid out 256 at a time
// (zeros for outliers: a sum that starts at 0 is unchanged by adding 0) and 45
// lanes accumulate the upper triangle of A^T A, each sequentially in match order.
__global__ __launch_bounds__(256) void fundamental_fit_kernel(const GeoImg* __restrict__ imgs,
                                                              const GeoPair* __restrict__ pairs,
                                                              const int32_t* __restrict__ match_idx,
                                                              const uint32_t* __restrict__ rnd, GeoParams prm,
                                                              GeoOut out, GeoFit* __restrict__ fits,
                                                              unsigned* __restrict__ err) {
    extern __shared__ __attribute__((aligned(16))) uint8_t dyn[];
    double* rows = reinterpret_cast<double*>(dyn);                            // [256][9]
    float4* pts = reinterpret_cast<float4*>(dyn + kGeoRowBytes);              // [cap]
    __shared__ double sF[9], s_sum[6];
    __shared__ uint32_t wtot[4];
    __shared__ unsigned long long s_best[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t p = blockIdx.x;
    const GeoPair pr = pairs[p];
    const GeoImg Q = imgs[pr.qi], T = imgs[pr.ti];

    // stage-1 matches, ascending query order
    uint32_t n = 0;
    for (int c0 = 0; c0 < Q.n; c0 += 256) {
        const int q = c0 + tid;
        int32_t m = q < Q.n ? match_idx[pr.out + q] : -1;
        if (m >= T.n) {
            atomicOr(err, 2u);
            m = -1;
        }
        uint32_t tot;
        const uint32_t pos = n + block_rank(m >= 0, wtot, &tot);
        if (m >= 0 && pos < (uint32_t)prm.cap)
            pts[pos] = make_float4(Q.kp[2 * q], Q.kp[2 * q + 1], T.kp[2 * m], T.kp[2 * m + 1]);
        n += tot;
    }
    // a pair that ends here: no matrix, nothing for the kernels that follow
    auto finish = [&](int st, int bh) {
        if (tid < 9) out.F[9 * p + tid] = 0.0;
        if (tid == 0) {
            out.n_matches[p] = (int32_t)n;
            out.n_inliers[p] = 0;
            out.best_h[p] = bh;
            out.status[p] = st;
            fits[p].refit = 0;
        }
    };
    if (n > (uint32_t)prm.cap) {
        if (tid == 0) atomicOr(err, 4u);
        finish(kDegenerate, -1);
        return;
    }
    if ((int)n < prm.min_matches || n < 8) {
        finish(kFewMatches, -1);
        return;
    }
    __syncthreads();

    // Hartley normalisation of both point sets (sequential sums)
    const double dn = (double)n;
    {
        const float* co = reinterpret_cast<const float*>(pts) + wv;  // this wave's coordinate
        double s = 0.0;
        for (uint32_t c0 = 0; c0 < n; c0 += 64) {
            const uint32_t i = c0 + (uint32_t)lane;
            s = add_lanes(s, i < n ? (double)co[4 * i] : 0.0, (int)min(64u, n - c0));
        }
        if (lane == 0) s_sum[wv] = s;
    }
    __syncthreads();
    const double cx = s_sum[0] / dn, cy = s_sum[1] / dn, cu = s_sum[2] / dn, cv = s_sum[3] / dn;
    if (wv < 2) {
        const double c0x = wv == 0 ? cx : cu, c0y = wv == 0 ? cy : cv;
        double s = 0.0;
        for (uint32_t c0 = 0; c0 < n; c0 += 64) {
            const uint32_t i = c0 + (uint32_t)lane;
            double v = 0.0;
            if (i < n) {
                const float4 m = pts[i];
                const double dx = (double)(wv == 0 ? m.x : m.z) - c0x, dy = (double)(wv == 0 ? m.y : m.w) - c0y;
                v = sqrt(dx * dx + dy * dy);
            }
            s = add_lanes(s, v, (int)min(64u, n - c0));
        }
        if (lane == 0) s_sum[4 + wv] = s;
    }
    __syncthreads();
    const double dq = s_sum[4], dt = s_sum[5];
    if (!(dq > 0.0 && dt > 0.0)) {
        finish(kDegenerate, -1);
        return;
    }
    const Norm2 NQ{kSqrt2 / (dq / dn), cx, cy}, NT{kSqrt2 / (dt / dn), cu, cv};
    const double dd = prm.thr * prm.thr;

    // hypotheses: pixel-space matrix of hypothesis h, false if unsolvable
    auto hypothesis = [&](int h, double (&Fh)[9]) -> bool {
        int idx[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = (int)n - 8 + i;
            int v = (int)(((uint64_t)rnd[8 * (size_t)h + i] * (uint64_t)(j + 1)) >> 32);
#pragma unroll
            for (int a = 0; a < i; ++a)
                if (idx[a] == v) v = j;
            idx[i] = v;
        }
        double A[8][9];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const float4 m = pts[idx[r]];
            design_row(nx(NQ, m.x), ny(NQ, m.y), nx(NT, m.z), ny(NT, m.w), A[r]);
        }
        double f[9];
        if (!null8(A, f)) return false;
        rank2(f);
        to_pixels(f, NQ, NT, Fh);
        return true;
    };
    int best_c = -1, best_h = 0x7FFFFFFF;
    for (int h = tid; h < prm.n_hyp; h += 256) {
        double Fh[9];
        if (!hypothesis(h, Fh)) continue;
        int cnt = 0;
        for (uint32_t i = 0; i < n; ++i) cnt += inlier(Fh, pts[i], dd) ? 1 : 0;
        if (cnt > best_c) {
            best_c = cnt;
            best_h = h;
        }
    }
    // block argmax of (count, -h); the winning thread rebuilds its matrix
    unsigned long long key = ((unsigned long long)(uint32_t)(best_c + 1) << 32) | (uint32_t)(0x7FFFFFFF - best_h);
    for (int d = 32; d >= 1; d >>= 1) {
        const unsigned long long o = __shfl_xor(key, d);
        key = o > key ? o : key;
    }
    if (lane == 0) s_best[wv] = key;
    __syncthreads();
    unsigned long long top = s_best[0];
    for (int w = 1; w < 4; ++w) top = s_best[w] > top ? s_best[w] : top;
    const int bc = (int)(top >> 32) - 1;
    const int bh = 0x7FFFFFFF - (int)(uint32_t)(top & 0xFFFFFFFFull);
    if (bc < 8) {
        finish(kDegenerate, bc >= 0 ? bh : -1);
        return;
    }
    if (best_h == bh) {
        double Fh[9];
        hypothesis(bh, Fh);
#pragma unroll
        for (int i = 0; i < 9; ++i) sF[i] = Fh[i];
    }
    __syncthreads();

    // refit: A^T A (upper triangle) over the best hypothesis's inliers
    double F[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) F[i] = sF[i];
    int r = 0, k = min(tid, 44);
    while (k >= 9 - r) {
        k -= 9 - r;
        ++r;
    }
    const int c = r + k;
    double acc = 0.0;
    for (uint32_t c0 = 0; c0 < n; c0 += 256) {
        const uint32_t i = c0 + (uint32_t)tid;
        double a[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) a[j] = 0.0;
        if (i < n) {
            const float4 m = pts[i];
            if (inlier(F, m, dd)) design_row(nx(NQ, m.x), ny(NQ, m.y), nx(NT, m.z), ny(NT, m.w), a);
        }
        __syncthreads();  // the last chunk's rows are read
#pragma unroll
        for (int j = 0; j < 9; ++j) rows[9 * tid + j] = a[j];
        __syncthreads();
        if (tid < 45) {
            const int cnt = (int)min(256u, n - c0);
#pragma unroll 8
            for (int i2 = 0; i2 < cnt; ++i2) acc = acc + rows[9 * i2 + r] * rows[9 * i2 + c];
        }
    }
    GeoFit& fit = fits[p];
    if (tid < 45) {
        fit.A[r * 9 + c] = acc;
        fit.A[c * 9 + r] = acc;
    }
    if (tid == 0) {
        fit.norm[0] = NQ.s;
        fit.norm[1] = NQ.cx;
        fit.norm[2] = NQ.cy;
        fit.norm[3] = NT.s;
        fit.norm[4] = NT.cx;
        fit.norm[5] = NT.cy;
        fit.refit = 1;
        out.n_matches[p] = (int32_t)n;
        out.best_h[p] = bh;
    }
}

// The smallest eigenvector of each pair's A^T A, made rank 2 and mapped to
// pixels.  27 lanes work on a pair, two pairs per wavefront: lane k on row k of
// A (the column step of a rotation), lane 9 + k on row k of V, lane 18 + k on
// column k of A (the row step); A and V lie in LDS.  The time is that of 360
// rotations one after another in a single wavefront: its instructions, of which
// the two square roots and three divisions of c and s are 95.  So the rest is
// kept short: a lane reads and writes two elements, the row step takes the
// block's column step in registers, the next rotation's c and s start from
// entries computed here and not from the LDS, and q is unrolled so that places
// are offsets: 124 instructions per rotation, 154 us at up to about 2000 pairs
// (nine lanes per pair, each doing a row's, V's and a column's work, 270
// instructions: 205 us).
constexpr int kRefitPairs = 2;
__global__ __launch_bounds__(64) void fundamental_refit_kernel(const GeoFit* __restrict__ fits, int64_t n_pairs,
                                                               GeoOut out) {
    __shared__ double s_M[kRefitPairs][2][81];  // A, then V
    const int lane = threadIdx.x;
    const int g = min(lane / 27, kRefitPairs - 1), kind = lane % 27 / 9, k = lane % 9;
    const int64_t p = (int64_t)blockIdx.x * kRefitPairs + g;
    const bool live = lane < 27 * kRefitPairs && p < n_pairs && fits[p].refit != 0;
    if (__ballot(live) == 0) return;
    double* A = s_M[g][0];
    double* V = s_M[g][1];
    if (live && kind < 2)
        for (int j = 0; j < 9; ++j) (kind == 0 ? A : V)[9 * k + j] = kind == 0 ? fits[p].A[9 * k + j] : j == k ? 1.0 : 0.0;
    wave_sync();
    // this lane's elements of a rotation (p, q): own[p * step], own[q * step]
    double* own = kind == 0 ? A + 9 * k : kind == 1 ? V + 9 * k : A + k;
    const int step = kind == 2 ? 9 : 1;
    // c and s of the rotation at hand; on: it is one (its entry is not 0)
    double c, s;
    bool on = live && A[1] != 0.0;
    schur(A[0], A[10], A[1], c, s);
    for (int sw = 0; sw < kJacobiSweeps9; ++sw)
#pragma unroll 1
        for (int pp = 0; pp < 8; ++pp) {
            const double* Arow = A + 9 * pp;  // A[pp][..]
            const double* Acol = A + pp;      // A[..][pp]
            double* mine = own + step * pp;
#pragma unroll
            for (int q = 1; q < 9; ++q) {
                if (q <= pp) continue;
                const double app = Arow[pp], apq = Arow[q], aqp = Acol[9 * q], aqq = A[10 * q];
                double u = *mine, v = own[step * q];
                // the next rotation's plane: (pp, q + 1), or (pp + 1, pp + 2)
                const int np = pp < 7 ? pp + 1 : 0;
                double n_pp = q < 8 ? 0.0 : A[10 * np], n_qq = q < 8 ? A[10 * q + 10] : A[10 * np + 10];
                double n_pq = q < 8 ? Arow[q + 1] : A[10 * np + 1];
                const double e = q < 8 ? A[10 * q + 1] : A[9 * np + pp];
                // the block after the column step
                const double bpp = c * app - s * apq, bpq = s * app + c * apq;
                const double bqp = c * aqp - s * aqq, bqq = s * aqp + c * aqq;
                if (q < 8) {
                    n_pp = on ? c * bpp - s * bqp : app;
                    const double w = c * n_pq - s * e;
                    n_pq = on ? w : n_pq;
                } else if (pp == 6) {  // (7, 8) follows (6, 8)
                    const double w = s * e + c * n_pq, z = s * bpq + c * bqq;
                    n_qq = on ? z : n_qq;
                    n_pq = on ? w : n_pq;
                }
                double c1, s1;
                schur(n_pp, n_qq, n_pq, c1, s1);
                const bool at_p = k == pp, at_q = k == q, row = kind == 2;
                u = row && at_p ? bpp : row && at_q ? bpq : u;
                v = row && at_p ? bqp : row && at_q ? bqq : v;
                const double nu = c * u - s * v, nv = s * u + c * v;
                if (on && (kind != 0 || (!at_p && !at_q))) {
                    *mine = nu;
                    own[step * q] = nv;
                }
                on = live && n_pq != 0.0;
                c = c1;
                s = s1;
                wave_sync();
            }
        }
    if (live && lane % 27 == 0) {
        int m = 0;
        for (int i = 1; i < 9; ++i)
            if (A[i * 9 + i] < A[m * 9 + m]) m = i;
        double f[9], F[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = V[i * 9 + m];
        rank2(f);
        const double* N = fits[p].norm;
        to_pixels(f, Norm2{N[0], N[1], N[2]}, Norm2{N[3], N[4], N[5]}, F);
#pragma unroll
        for (int i = 0; i < 9; ++i) out.F[9 * p + i] = F[i];
    }
}

// Inliers of the refit matrices and the pairs' status.
__global__ __launch_bounds__(256) void fundamental_count_kernel(const GeoImg* __restrict__ imgs,
                                                                const GeoPair* __restrict__ pairs,
                                                                const int32_t* __restrict__ match_idx, double thr,
                                                                const GeoFit* __restrict__ fits, GeoOut out) {
    __shared__ uint32_t wtot[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t p = blockIdx.x;
    if (fits[p].refit == 0) return;
    const GeoPair pr = pairs[p];
    const GeoImg Q = imgs[pr.qi], T = imgs[pr.ti];
    const double dd = thr * thr;
    double F[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) F[i] = out.F[9 * p + i];
    uint32_t cnt = 0;
    for (int q = tid; q < Q.n; q += 256) {
        const int32_t m = match_idx[pr.out + q];
        if (m >= 0 && m < T.n)
            cnt += inlier(F, make_float4(Q.kp[2 * q], Q.kp[2 * q + 1], T.kp[2 * m], T.kp[2 * m + 1]), dd) ? 1u : 0u;
    }
    for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d);
    if (lane == 0) wtot[wv] = cnt;
    __syncthreads();
    if (tid == 0) {
        const int ni = (int)(wtot[0] + wtot[1] + wtot[2] + wtot[3]);
        out.n_inliers[p] = ni;
        out.status[p] = 3ll * ni >= 2ll * (long long)out.n_matches[p] ? kAccept : kFewInliers;
    }
}

hipError_t launch_top_scale(hipStream_t s, const SelectImg* imgs, int n_images) {
    if (n_images <= 0) return hipSuccess;
    hipLaunchKernelGGL(top_scale_kernel, dim3(n_images), dim3(256), 0, s, imgs);
    return hipGetLastError();
}

hipError_t launch_gather_rows(hipStream_t s, const GatherImg* imgs, const RowChunk* chunks, int n_chunks,
                              unsigned* err) {
    if (n_chunks <= 0) return hipSuccess;
    const int grid = n_chunks < 65536 ? n_chunks : 65536;
    hipLaunchKernelGGL(gather_rows_kernel, dim3(grid), dim3(256), 0, s, imgs, chunks, n_chunks, err);
    return hipGetLastError();
}

size_t fundamental_lds_bytes(int cap) { return kGeoRowBytes + (size_t)cap * 16; }

hipError_t launch_fundamental(hipStream_t s, const GeoImg* imgs, const GeoPair* pairs, int64_t n_pairs,
                              const int32_t* match_idx, const uint32_t* rnd, const GeoParams& prm, const GeoOut& out,
                              GeoFit* fits, unsigned* err) {
    if (n_pairs <= 0) return hipSuccess;
    const size_t lds = (fundamental_lds_bytes(prm.cap) + 15) & ~size_t(15);
    if (lds > 65536) {
        // dynamic LDS beyond 64 KB has to be allowed explicitly
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&fundamental_fit_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    CH_LAUNCH(fundamental_fit_kernel, dim3((unsigned)n_pairs), dim3(256), lds, s, imgs, pairs, match_idx, rnd, prm, out,
              fits, err);
    CH_LAUNCH(fundamental_refit_kernel, dim3((unsigned)((n_pairs + kRefitPairs - 1) / kRefitPairs)), dim3(64), 0, s, fits,
              n_pairs, out);
    CH_LAUNCH(fundamental_count_kernel, dim3((unsigned)n_pairs), dim3(256), 0, s, imgs, pairs, match_idx, prm.thr, fits,
              out);
    return hipSuccess;
}

}  // namespace cashash
