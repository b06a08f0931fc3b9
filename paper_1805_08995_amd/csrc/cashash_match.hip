// The CasHash matcher for gfx950 (MI355X): "Review of Cascade Hashing",
// Steps 1-4, "Improved Parallel Hashing Ranking" and Eq. 1-2.
//
// One wavefront per tile of up to 32 consecutive queries of one pair.  Train
// images are pre-sorted into per-table buckets whose entries carry code, keys
// and index, so a query's candidates are six contiguous runs read 64 at a
// time.  Candidates whose key (Hamming << 16 | index) is at most a threshold
// carried from query to query go to a short list in LDS; the k smallest of the
// list are found from the paper's index table (a histogram over Hamming
// distance, scanned with DPP) and ties at the k-th distance are broken by
// index.  The tile's kept candidates are measured with v_dot4_u32_u8 (exact),
// then the ratio test runs one lane per query.  All pairs run in one persistent
// launch (two when small and large train images meet) with per-XCD work
// segments.
#include "cashash_device.h"
#include "cashash_launch.h"

namespace cashash {

// ------------------------------------------------------------------ matching

// x as seen through a DPP pattern; lanes whose source is outside their row,
// or whose row is masked off, receive 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
    return __builtin_amdgcn_update_dpp(0u, x, CTRL, ROW_MASK, 0xf, false);
}

// Inclusive prefix sum over the 64 lanes with DPP row shifts and row
// broadcasts (no LDS round trip).
__device__ __forceinline__ uint32_t wave_scan_dpp(uint32_t x) {
    x += dpp<0x111, 0xf>(x);  // row_shr:1
    x += dpp<0x112, 0xf>(x);  // row_shr:2
    x += dpp<0x114, 0xf>(x);  // row_shr:4
    x += dpp<0x118, 0xf>(x);  // row_shr:8
    x += dpp<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
    x += dpp<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
    return x;
}

__device__ __forceinline__ uint32_t readlane(uint32_t v, int l) { return __builtin_amdgcn_readlane(v, l); }

// popcount(x) + acc as one v_bcnt_u32_b32 (a dependent chain keeps the
// compiler from splitting a 128-bit count into two halves and an add).
__device__ __forceinline__ uint32_t bcnt_acc(uint32_t x, uint32_t acc) {
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

// popcount(x) by the same instruction.
__device__ __forceinline__ uint32_t bcnt(uint32_t x) {
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, 0" : "=v"(r) : "v"(x));
    return r;
}

// ------------------------------------------------------------------ shared by both matcher kernels

// Arguments needed only when work is grabbed or a tile is finished, kept in
// LDS rather than in scalar registers (the kernels are short of them), and the
// block's sums of the statistics.
struct Rare {
    int32_t* o_idx;
    int32_t* o_d1;
    int32_t* o_d2;
    uint32_t* ctl;
    int64_t num2, den2;
    int32_t seg[kSegments + 1];
    int32_t grab, set;
    uint32_t done, empty;  // wavefronts that ended; exhausted segments
    unsigned long long sum[3];
    __device__ __forceinline__ void fill(const MatchParams& prm, uint32_t* c, int32_t* idx, int32_t* d1, int32_t* d2) {
        o_idx = idx;
        o_d1 = d1;
        o_d2 = d2;
        ctl = c;
        num2 = prm.num2;
        den2 = prm.den2;
        for (int i = 0; i <= kSegments; ++i) seg[i] = prm.seg[i];
        grab = prm.grab;
        set = prm.set;
        done = empty = 0;
        sum[0] = sum[1] = sum[2] = 0;
    }
    __device__ __forceinline__ uint32_t* counter(uint32_t x) const { return ctl + x * kCtlStride + set; }
    // A wavefront's statistics at its end (lane 0): bucket entries, union
    // sizes, ranked.  The block's last wavefront adds the block's sums to one
    // of kStatSlots places: atomics of every wavefront on the same three words
    // had queued for 0.3 ms a launch.
    __device__ __forceinline__ void add_stats(uint64_t bucket, uint64_t uni, uint64_t ranked) {
        atomicAdd(&sum[0], (unsigned long long)bucket);
        atomicAdd(&sum[1], (unsigned long long)uni);
        atomicAdd(&sum[2], (unsigned long long)ranked);
        __threadfence_block();
        if (atomicAdd(&done, 1u) != (uint32_t)kWavesPerBlock - 1u) return;
        unsigned long long* s = stat_slot(ctl, (int)(blockIdx.x % kStatSlots));
        for (int i = 0; i < 3; ++i) {
            const unsigned long long v = atomicAdd(&sum[i], 0ull);
            if (v) atomicAdd(s + i, v);
        }
    }
};

// A persistent wavefront's share of the work list: it takes `grab` items at a
// time from its own XCD's segment (blocks are placed on the XCDs in turn),
// whose train images stay in that XCD's L2, and moves to the other segments
// when that one is exhausted.  A segment found exhausted is noted for the whole
// block, so that at the end of a launch a counter is asked once per block and
// not by each of up to 8192 wavefronts.
struct Grab {
    int32_t cur = 0, end = 0;
    // false: every segment is exhausted
    __device__ __forceinline__ bool next(Rare& rare, int lane, int32_t& it) {
        if (cur >= end) {
#pragma unroll 1
            for (int sx = 0; sx < kSegments; ++sx) {
                const uint32_t x = (blockIdx.x + (uint32_t)sx) & (kSegments - 1);
                const int32_t s0 = rare.seg[x], s1 = rare.seg[x + 1];
                if (s0 >= s1 || ((rare.empty >> x) & 1u)) continue;
                uint32_t v = 0;
                const int32_t n = rare.grab;
                if (lane == 0) v = atomicAdd(rare.counter(x), (uint32_t)n);
                v = readlane(v, 0);
                if ((int64_t)s0 + v < (int64_t)s1) {
                    cur = s0 + (int32_t)v;
                    end = min(cur + n, s1);
                    break;
                }
                if (lane == 0) atomicOr(&rare.empty, 1u << x);
            }
            if (cur >= end) return false;
        }
        it = cur++;
        return true;
    }
};

// Step 4 and the ratio test of one tile of nq <= kMaxTile queries.  sel: the
// train indices kept, query by query; lane l's `kept` is query l's kept count
// and first place in sel (<< 16).  Four lanes take one query at a time (lanes
// 4g .. the queries R g + r, r = 0 .. R - 1): they hold its descriptor and go
// through its candidates with v_dot4_u32_u8 (exact), so that a query's row is
// loaded once, and each load of the four lanes is 64 consecutive bytes of one
// row, one L1 access.  Every lane of the four ends with the nearest and second
// nearest; lane 4g + r keeps those of round r.
__device__ __forceinline__ void finish_tile(int lane, int nq, int32_t q0, const uint8_t* __restrict__ qdesc,
                                            const uint8_t* __restrict__ tdesc, int64_t out, uint32_t kept,
                                            const uint16_t* sel, const Rare& rare) {
    asm volatile("" : "+v"(lane));  // what follows from it is worked out here, not kept from tile to tile
    const int g = lane >> 2, part = lane & 3;
    const int R = (nq + 15) >> 4;
    const uint32_t part16 = (uint32_t)part << 4;
    // a row's bytes 16 part .. and 64 + 16 part ..
    struct Row {
        uint4 lo, hi;
    };
    auto row = [&](const uint8_t* base, uint32_t i) {
        const uint32_t at = (i << 7) + part16;
        return Row{gload(reinterpret_cast<const uint4*>(base + at)), gload(reinterpret_cast<const uint4*>(base + at + 64))};
    };
    auto dot = [](const Row& x, const Row& y, uint32_t c) {
        c = __builtin_amdgcn_udot4(x.lo.x, y.lo.x, c, false);
        c = __builtin_amdgcn_udot4(x.lo.y, y.lo.y, c, false);
        c = __builtin_amdgcn_udot4(x.lo.z, y.lo.z, c, false);
        c = __builtin_amdgcn_udot4(x.lo.w, y.lo.w, c, false);
        c = __builtin_amdgcn_udot4(x.hi.x, y.hi.x, c, false);
        c = __builtin_amdgcn_udot4(x.hi.y, y.hi.y, c, false);
        c = __builtin_amdgcn_udot4(x.hi.z, y.hi.z, c, false);
        return __builtin_amdgcn_udot4(x.hi.w, y.hi.w, c, false);
    };
    auto sum4 = [](uint32_t d) {
        d += dpp<0xB1, 0xf>(d);         // quad_perm [1,0,3,2]
        return d + dpp<0x4E, 0xf>(d);   // quad_perm [2,3,0,1]
    };
    int32_t f_d1 = 0, f_d2 = 0;
    uint32_t f_j = 0, f_n = 0;
    for (int r = 0; r < R; ++r) {
        const int q = min(R * g + r, nq - 1);
        const uint32_t kw = (uint32_t)__shfl((int)kept, q);
        const uint32_t n = kw & 0xFFFFu;
        const uint16_t* my = sel + (kw >> 16);
        const Row av = row(qdesc, (uint32_t)(q0 + q));
        // |b|^2 - 2 a.b of a candidate's row: the distance less |a|^2
        auto rel = [&](const Row& b) {
            return (int32_t)sum4(dot(b, b, (uint32_t)__mul24((int)dot(av, b, 0u), -2)));
        };
        int32_t best = INT32_MAX, sec = INT32_MAX;
        uint32_t bj = 0;
        auto take = [&](int32_t d, uint32_t j) {
            sec = max(min(d, sec), min(best, max(d, sec)));  // the middle one of d, best <= sec
            bj = d < best ? j : bj;
            best = min(best, d);
        };
        // two candidates at a time while every query of the round has two
        // more, then one at a time
        uint32_t s = 0;
        for (; __builtin_amdgcn_ballot_w64(s + 2 > n) == 0; s += 2) {
            const uint32_t j0 = my[s], j1 = my[s + 1];
            const Row b0 = row(tdesc, j0), b1 = row(tdesc, j1);
            take(rel(b0), j0);
            take(rel(b1), j1);
        }
        for (; __builtin_amdgcn_ballot_w64(s < n) != 0; ++s)
            if (s < n) {
                const uint32_t j = my[s];
                take(rel(row(tdesc, j)), j);
            }
        // equal nearest and second: the smallest index among the nearest
        if (__builtin_amdgcn_ballot_w64(best == sec && n > 1) != 0)
            for (s = 0; __builtin_amdgcn_ballot_w64(s < n) != 0; ++s)
                if (s < n) {
                    const uint32_t j = my[s];
                    if (rel(row(tdesc, j)) == best) bj = min(bj, j);
                }
        const int32_t aa = (int32_t)sum4(dot(av, av, 0u));
        if (part == r) {
            f_d1 = best + aa;
            f_d2 = sec + aa;
            f_j = bj;
            f_n = n;
        }
    }
    if (part < R && R * g + part < nq) {
        int32_t r_idx = -1, r_d1 = -1, r_d2 = -1;
        if (f_n >= 1) r_d1 = f_d1;
        if (f_n >= 2) {
            r_d2 = f_d2;
            if (rare.den2 * (int64_t)r_d1 < rare.num2 * (int64_t)r_d2) r_idx = (int32_t)f_j;
        }
        const int64_t o = out + q0 + R * g + part;
        gstore(rare.o_idx + o, r_idx);
        gstore(rare.o_d1 + o, r_d1);
        gstore(rare.o_d2 + o, r_d2);
    }
    wave_sync();
}

// ------------------------------------------------------------------ plain form

// Inclusive rank structure of one query's six bucket runs in LDS (kRunWords +
// 2 NC words per query, written by the tile setup), for the runs concatenated
// in table order:
//   words 2o, 2o+1  : of the o-th non-empty run (table t), the byte offset that
//                     takes candidate e's 16 e to its entry's code, 16 (t n +
//                     b_t - start), and the query's keys as table t's entries
//                     are compared with them (see first_seen)
//   words 12 ..     : per 64-candidate chunk u < NC the 64-bit mask of run
//                     starts (bit j: a run other than the first starts at
//                     candidate 64u + j + 1), so that a lane counts the starts
//                     at or below its candidate, its run's ordinal, with mbcnt
constexpr int kRunWords = 12;

// Candidates kept per query on the way to its k nearest: at most kPassCap keys
// pass the threshold, read back as up to three per lane.
constexpr int kPassCap = 192;
constexpr int kPassSlots = kPassCap / 64;
// Keys the list in LDS holds, in front of select_64's histogram.
constexpr int kListKeys = 256;

// Entry word `kw` (see bucket_kernel) against the query's: the lanes whose
// candidate shares no key of an earlier table with the query (one that does
// is in that table's run already).  Bytes 0-3: the entry holds 0 in the bytes
// of its own and later tables and the query word 0xFF there, so a zero byte of
// the difference is a shared key of an earlier table.  Key 4 only matters to
// table 5's entries; the others hold 0x100 in its 16 bits, which no key equals.
__device__ __forceinline__ uint64_t first_seen(uint2 kw, uint32_t qlo, uint32_t q4) {
    const uint32_t y = kw.x ^ qlo;
    // bitop3 truth table 0x20 = a & ~b & c: the exact zero-byte test
    const uint32_t z = __builtin_amdgcn_bitop3_b32(y - 0x01010101u, y, 0x80808080u, 0x20);
    return __builtin_amdgcn_ballot_w64(z == 0u) & __builtin_amdgcn_ballot_w64((uint16_t)kw.y != (uint16_t)q4);
}

// The loads of C chunks of 64 candidates, all in flight together, then each
// chunk's keys (Hamming << 16 | index) and whether the lane's candidate is a
// valid one (inside the runs and not a repeat).  ORD: positions by the chunk
// start masks (chunk u0 + c < NC); else by comparing with the run starts P.
// Lanes past the last run neither load nor are valid.
template <int C, bool ORD>
struct Chunks {
    uint32_t key[C];
    uint64_t ok[C];  // lane masks
    __device__ __forceinline__ void load(int lane, const char* code, const char* kid, const uint32_t* qrow, int u0,
                                         uint32_t preq, const uint32_t (&P)[5], uint32_t total,
                                         const uint32_t (&qc)[4]) {
        uint2 run[C];
        uint32_t off[C];
        const uint32_t lane16 = (uint32_t)lane << 4;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            uint32_t o;
            if constexpr (ORD) {
                const uint2 sm = *reinterpret_cast<const uint2*>(qrow + kRunWords + 2 * (u0 + c));
                const uint32_t o0 = (preq >> (3 * (u0 + c))) & 7u;
                o = __builtin_amdgcn_mbcnt_hi(sm.y, __builtin_amdgcn_mbcnt_lo(sm.x, o0));
            } else {
                const uint32_t e = 64u * (uint32_t)(u0 + c) + (uint32_t)lane;
                o = (uint32_t)(e >= P[0]) + (e >= P[1]) + (e >= P[2]) + (e >= P[3]) + (e >= P[4]);
            }
            run[c] = *reinterpret_cast<const uint2*>(qrow + 2 * o);
            off[c] = run[c].x + lane16;
        }
        ulonglong2 cd[C];
        uint2 kw[C];
        const char* cb = code + 1024 * u0;
        const char* kb = kid + 512 * u0;
        // the last chunk's lanes inside the runs; only they load (the empty asm
        // keeps every case's mask from being computed ahead of the switch)
        int tot = (int)total;
        asm volatile("" : "+s"(tot));
        const uint64_t live = ~0ull >> max(64 * (u0 + C) - tot, 0);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (c + 1 < C || __builtin_amdgcn_inverse_ballot_w64(live)) {
                cd[c] = gload(reinterpret_cast<const ulonglong2*>(cb + off[c] + 1024 * c));
                kw[c] = gload(reinterpret_cast<const uint2*>(kb + (off[c] >> 1) + 512 * c));
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            uint32_t h = bcnt((uint32_t)cd[c].x ^ qc[0]);
            h = bcnt_acc((uint32_t)(cd[c].x >> 32) ^ qc[1], h);
            h = bcnt_acc((uint32_t)cd[c].y ^ qc[2], h);
            h = bcnt_acc((uint32_t)(cd[c].y >> 32) ^ qc[3], h);
            key[c] = __builtin_amdgcn_alignbyte(h, kw[c].y, 2);  // h << 16 | index
            ok[c] = first_seen(kw[c], run[c].y, preq >> 24);
            if (c + 1 == C) ok[c] &= live;
        }
    }
};

// Place of this lane, one of the mask's, behind the first n words of a list
// (added to the list's address rather than to the count: one scalar operand
// per instruction).
template <class T>
__device__ __forceinline__ T& list_at(T* list, uint32_t n, uint64_t m) {
    return (list + n)[mbcnt64(m)];
}

// The same with the keys that pass the threshold (key <= K) appended to the
// LDS list and counted in n_pass; n_union counts the valid candidates.
template <int C, bool ORD>
__device__ __forceinline__ void scan_chunks(int lane, const char* code, const char* kid, const uint32_t* qrow, int u0,
                                            uint32_t preq, const uint32_t (&P)[5], uint32_t total,
                                            const uint32_t (&qc)[4], uint32_t K, uint32_t* list, uint32_t& n_pass,
                                            uint32_t& n_union) {
    Chunks<C, ORD> ch;
    ch.load(lane, code, kid, qrow, u0, preq, P, total, qc);
#pragma unroll
    for (int c = 0; c < C; ++c) {
        n_union += (uint32_t)__popcll(ch.ok[c]);
        const uint64_t m = ch.ok[c] & __builtin_amdgcn_ballot_w64(ch.key[c] <= K);
        if (__builtin_amdgcn_inverse_ballot_w64(m)) list_at(list, n_pass, m) = ch.key[c];
        n_pass += (uint32_t)__popcll(m);
    }
}

// The n listed keys, S registers per lane (~0u past them).
template <int S>
__device__ __forceinline__ void read_list(uint32_t (&r)[S], const uint32_t* list, uint32_t n, int lane) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const uint32_t v = list[64 * s + lane];
        r[s] = 64u * s + (uint32_t)lane < n ? v : ~0u;
    }
}

// A bound that exactly the kk smallest of the n keys r (all <= K, distinct,
// n > kk >= 1) are within.  Step 3: the Hamming distance H* of the kk-th by
// counting with ballots from the previous query's H* (hG), ties there by index.
template <int S>
__device__ __forceinline__ uint32_t kth_bound(const uint32_t (&r)[S], uint32_t n, uint32_t K, uint32_t kk,
                                              int32_t& hG) {
    auto count = [&](uint32_t x) {  // keys <= x
        uint32_t c = 0;
#pragma unroll
        for (int s = 0; s < S; ++s) c += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(r[s] <= x));
        return c;
    };
    auto upto = [](int32_t h) { return ((uint32_t)h << 16) | 0xFFFFu; };
    int32_t lo = -1, hi = (int32_t)(K >> 16), step = 2;
    uint32_t chi = n;  // keys of Hamming distance <= hi; fewer than kk at lo
    const int32_t g = min(hG, hi - 1);
    if (g >= 0) {
        uint32_t c = count(upto(g));
        if (c >= kk) {
            hi = g;
            chi = c;
            while (hi - step > lo) {
                c = count(upto(hi - step));
                if (c < kk) {
                    lo = hi - step;
                    break;
                }
                hi -= step;
                chi = c;
                step += step;
            }
        } else {
            lo = g;
            while (lo + step < hi) {
                c = count(upto(lo + step));
                if (c >= kk) {
                    hi = lo + step;
                    chi = c;
                    break;
                }
                lo += step;
                step += step;
            }
        }
    }
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        const uint32_t c = count(upto(mid));
        if (c >= kk) {
            hi = mid;
            chi = c;
        } else {
            lo = mid;
        }
    }
    hG = hi;
    const uint32_t top = min(K, upto(hi));
    if (chi == kk) return top;
    // more at H* than needed: the bound with exactly kk keys within it (the
    // keys are distinct, so the count goes through kk), key by key if few are
    // there, else by halves over the indices
    const uint32_t at = (uint32_t)hi << 16;
    if (chi - kk < 8u) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            uint64_t m = __builtin_amdgcn_ballot_w64(r[s] >= at) & __builtin_amdgcn_ballot_w64(r[s] <= top);
            while (m != 0) {
                const uint32_t x = readlane(r[s], __ffsll((unsigned long long)m) - 1);
                if (count(x) == kk) return x;
                m &= m - 1;
            }
        }
    } else {
        uint32_t from = at, to = top;
        while (from < to) {
            const uint32_t mid = from + ((to - from) >> 1);
            const uint32_t c = count(mid);
            if (c == kk) return mid;
            if (c < kk)
                from = mid + 1u;
            else
                to = mid;
        }
    }
    return max(at, 1u) - 1u;
}

// The kk smallest of the n listed keys (all <= K, distinct, n >= kk >= 1, S
// registers per lane): their indices appended to the tile list.
template <int S>
__device__ __forceinline__ void select_keys(const uint32_t* list, uint32_t n, uint32_t K, uint32_t kk, int lane,
                                            uint16_t* sel, uint32_t& sel_n, int32_t& hG) {
    uint32_t r[S];
    read_list(r, list, n, lane);
    const uint32_t tkey = n > kk ? kth_bound(r, n, K, kk, hG) : K;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const bool keep = r[s] <= tkey;
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
        if (keep) list_at(sel, sel_n, m) = (uint16_t)r[s];
        sel_n += (uint32_t)__popcll(m);
    }
}

// The list brought down to the kk smallest of its n > kk keys (S registers per
// lane); K: the bound that keys yet to come must be within.
template <int S>
__device__ __forceinline__ void shorten_list(uint32_t* list, uint32_t& n, uint32_t& K, uint32_t kk, int lane,
                                             int32_t& hG) {
    uint32_t r[S];
    wave_sync();
    read_list(r, list, n, lane);
    K = kth_bound(r, n, K, kk, hG);
    wave_sync();
    n = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const bool keep = r[s] <= K;
        const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
        if (keep) list_at(list, n, m) = r[s];
        n += (uint32_t)__popcll(m);
    }
}

// select_keys for at most 64 listed keys, one per lane: H* from a histogram
// over the 64 Hamming distances around the last H* (the paper's index table;
// hist: 64 cleared words of LDS, left cleared), scanned with DPP.  An H* at
// the ends of that window takes the counting form above.
__device__ __forceinline__ void select_64(const uint32_t* list, uint32_t* hist, uint32_t n, uint32_t K, uint32_t kk,
                                          int lane, uint16_t* sel, uint32_t& sel_n, int32_t& hG) {
    const uint32_t v = list[lane];
    const uint32_t r = (uint32_t)lane < n ? v : ~0u;
    uint32_t tkey = K;
    if (n > kk) {
        const int32_t base = hG - 32;
        const int32_t bin = min(max((int32_t)(r >> 16) - base, 0), 63);
        if ((uint32_t)lane < n) atomicAdd(hist + bin, 1u);
        wave_sync();
        const uint32_t incl = wave_scan_dpp(hist[lane]);
        hist[lane] = 0u;
        const uint64_t reach = __builtin_amdgcn_ballot_w64(incl >= kk);
        int L = __builtin_ctzll(reach);  // some bin reaches kk: n > kk
        asm("" : "+s"(L));               // a 32-bit value: the compare below stays scalar
        if ((uint32_t)(L - 1) >= 62u) {
            select_keys<1>(list, n, K, kk, lane, sel, sel_n, hG);
            return;
        }
        hG = base + L;
        const uint32_t at = (uint32_t)hG << 16;
        tkey = at | 0xFFFFu;
        if (readlane(incl, L) > kk) {
            // more at H* than needed: the one with exactly kk keys up to it
            uint64_t m = __builtin_amdgcn_ballot_w64(r >= at) & __builtin_amdgcn_ballot_w64(r <= tkey);
            tkey = max(at, 1u) - 1u;
            while (m != 0) {
                const int l = __builtin_ctzll(m);
                const uint32_t x = readlane(r, l);
                if ((uint32_t)__popcll(__builtin_amdgcn_ballot_w64(r <= x)) == kk) {
                    tkey = x;
                    break;
                }
                m ^= 1ull << l;
            }
        }
    }
    const bool keep = r <= tkey;
    const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
    if (keep) list_at(sel, sel_n, m) = (uint16_t)r;
    sel_n += (uint32_t)__popcll(m);
}

// The run starts of a lane's query (~0u: no run, or the first one), needed only
// past the chunk masks: one word each, or as halves of three words for trains
// whose starts fit 16 bits (NC == 4: at most 6 kLargeTrain entries).
template <int NC>
constexpr int kStartWords = NC == 4 ? 3 : 5;
static_assert(kTables * kLargeTrain < 0xFFFF, "run starts fit 16 bits");
template <int W>
__device__ __forceinline__ void put_start(uint32_t (&v)[W], int i, uint32_t start) {
    if constexpr (W == 5)
        v[i] = start;
    else
        v[i >> 1] = i & 1 ? v[i >> 1] | (start << 16) : start & 0xFFFFu;
}
template <int W>
__device__ __forceinline__ void run_starts(uint32_t (&P)[5], const uint32_t (&v)[W], int qi) {
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        if constexpr (W == 5)
            P[i] = readlane(v[i], qi);
        else
            P[i] = i & 1 ? readlane(v[i >> 1], qi) >> 16 : readlane(v[i >> 1], qi) & 0xFFFFu;
    }
}

// The plain form.  Per query: the six runs' candidates in 64-wide chunks, up to
// four chunks' loads in flight together, the keys that pass the threshold to
// the LDS list, then the selection.  A threshold that lets fewer than k pass is
// raised and the runs are read again (at most twice per query: six bits wider,
// then without a threshold; none of 2000 queries among 8000 points at k = 10,
// 3.5% at k = 40, 1.9% at k = 64); a list that gets full is brought down to its
// k smallest keys on the way, so crowded distances cost no second reading.  So no
// candidate is kept in a register past its chunk, the number of chunks has no
// limit, and the ranking works on one register per lane instead of one per
// chunk.  NC: chunks with start masks.
//
// What bounds it (100 x 8000 points, rocprofv3): issue.  Per query 153 VALU and
// 134 SALU instructions (213 and 132 when every candidate was kept in registers,
// ranked by an index table over all of them and compacted from them), 0.83 and
// 0.74 of the pipes' rates, and 61 L2 lines, 26 of the 29 TB/s that a plain read
// of such runs gets from L2 here.  Against that form: 100 x 8000 points 15.4 ->
// 11.8 ms, 16 x 20000 3.88 -> 1.77 ms per call (half of its queries had more
// candidates than its eight registers).  Crowded distances, 12 x 8000 points of which 250 /
// 600 / 3000 are equal: 0.37 / 0.58 / 4.6 ms, of which the widest bucket runs are
// most (with the threshold moved down by rereading 0.61 / 1.1 / 8.6; every
// candidate in registers or a list 0.57 / 4.0 / 71).
// The 4-slot form's eight blocks leave 64 registers: the wavefront's count of
// bucket entries lies in scratch, read and written once per tile (the launch
// writes 0.34 GB more than its 0.48 GB of outputs; with seven blocks there is
// no scratch and 60 x 8000 points take 3% longer, see match_blocks_per_cu).
template <int NC>
__global__ __launch_bounds__(256, match_blocks_per_cu(false, NC)) void plain_match_kernel(
    const ImgDev* __restrict__ imgs, const PairDev* __restrict__ pairs, const Item* __restrict__ items,
    int32_t n_items, uint32_t* __restrict__ ctl, MatchParams prm, int32_t* __restrict__ o_idx,
    int32_t* __restrict__ o_d1, int32_t* __restrict__ o_d2) {
    constexpr int kQS = kRunWords + 2 * NC;
    __shared__ __attribute__((aligned(16))) uint32_t s_list[kWavesPerBlock][kListKeys + 64];
    __shared__ __attribute__((aligned(16))) uint16_t s_sel[kWavesPerBlock][kSelCap];
    __shared__ __attribute__((aligned(16))) uint32_t s_qtab[kWavesPerBlock][kMaxTile * kQS];
    __shared__ Rare s_rare;
    if (threadIdx.x == 0) s_rare.fill(prm, ctl, o_idx, o_d1, o_d2);
    __syncthreads();
    const bool persistent = prm.grab > 0;
    const int lane = threadIdx.x & 63;
    const int wv = (int)uniform(threadIdx.x >> 6);
    uint32_t* list = s_list[wv];
    uint32_t* hist = list + kListKeys;
    uint16_t* sel = s_sel[wv];
    uint32_t* qtab = s_qtab[wv];
    hist[lane] = 0u;
    uint64_t st_bucket = 0, st_ranked = 0;  // per lane
    uint64_t st_union = 0;                   // uniform
    const uint32_t tauK = ((uint32_t)prm.tau << 16) | 0xFFFFu;
    uint32_t hK = min(tauK, (56u << 16) | 0xFFFFu);  // threshold for the next query
    int32_t hG = 52;                                  // the last query's H*

    Grab grab;
    int32_t it = (int32_t)(blockIdx.x * kWavesPerBlock + wv);
    for (;;) {
        if (persistent && !grab.next(s_rare, lane, it)) break;
        if (it >= n_items) break;
        const Item item = items[it];
        const PairDev& pr = pairs[item.pair];
        const ImgDev Q = imgs[pr.qi];
        const ImgDev T = imgs[pr.ti];
        const char* code = reinterpret_cast<const char*>(T.ent);
        const char* kid = code + (size_t)kTables * T.n * 16;
        const int nq = (int)uniform((uint32_t)item.nq);
        const int32_t q0 = (int32_t)uniform((uint32_t)item.q0);

        // ---- setup, one lane per query of the tile
        uint32_t v_P[kStartWords<NC>], v_total, v_preq;
        uint4 v_code;
        {
            const int64_t lq = q0 + min(lane, nq - 1);
            // (8-byte aligned)
            const uint2 c0 = gload(reinterpret_cast<const uint2*>(Q.codes + 2 * lq));
            const uint2 c1 = gload(reinterpret_cast<const uint2*>(Q.codes + 2 * lq + 1));
            v_code = make_uint4(c0.x, c0.y, c1.x, c1.y);
            const uint16_t* kq = reinterpret_cast<const uint16_t*>(Q.keys + 6 * lq);
            const uint32_t k01 = gload(kq), k23 = gload(kq + 1), k45 = gload(kq + 2);
            const uint32_t qlo = k01 | (k23 << 16);
            uint32_t b[kTables], e[kTables];
#pragma unroll
            for (int t = 0; t < kTables; ++t) {
                const uint32_t v = ((t < 4 ? qlo >> (8 * t) : k45 >> (8 * (t - 4)))) & 0xFFu;
                b[t] = gload(T.off + t * kOffStride + v);
                e[t] = gload(T.off + t * kOffStride + v + 1);
            }
            uint32_t* qt = qtab + kQS * lane;
            const bool own = lane < kMaxTile;
            if (own) {
#pragma unroll
                for (int i = 0; i < NC / 2; ++i)
                    reinterpret_cast<uint4*>(qt + kRunWords)[i] = make_uint4(0u, 0u, 0u, 0u);
            }
            uint32_t acc = 0, cnt = 0;  // entries and non-empty runs before table t
            uint32_t pre = 0;           // run starts at or below 64u, at bits 3u
#pragma unroll
            for (int t = 0; t < kTables; ++t) {
                const uint32_t len = e[t] - b[t];
                const bool inner = len != 0 && cnt != 0;  // a run start after the first
                if (t > 0) put_start(v_P, t - 1, inner ? acc : ~0u);
                if (own && len != 0)
                    *reinterpret_cast<uint2*>(qt + 2 * cnt) =
                        make_uint2(((uint32_t)t * (uint32_t)T.n + b[t] - acc) << 4, t < 4 ? qlo | (~0u << (8 * t)) : qlo);
                if (own && inner && acc <= 64u * NC)
                    atomicOr(qt + kRunWords + ((acc - 1u) >> 5), 1u << ((acc - 1u) & 31u));
#pragma unroll
                for (int u = 1; u < NC; ++u) pre += (uint32_t)(inner && acc <= 64u * u) << (3 * u);
                cnt += len != 0;
                acc += len;
            }
            if (lane < nq) st_bucket += acc;
            v_total = acc;
            v_preq = pre | (k45 << 24);  // and key 4 above it
            wave_sync();
        }
        uint32_t sel_n = 0;
        uint32_t v_kept = 0;  // lane qi: its kept count and first tile-list slot
        uint32_t t_union = 0;

        for (int qi = 0; qi < nq; ++qi) {
            // from lane qi (a load at a wave-uniform address would take as many
            // L1 accesses as one of 64 codes)
            const uint32_t qc[4] = {readlane(v_code.x, qi), readlane(v_code.y, qi), readlane(v_code.z, qi),
                                    readlane(v_code.w, qi)};
            const uint32_t total = readlane(v_total, qi), preq = readlane(v_preq, qi);
            const uint32_t* qrow = qtab + kQS * qi;
            uint32_t K = total > 64u ? hK : tauK;  // a single chunk fits the list whole
            uint32_t n_pass = 0, n_union = 0;
            const uint32_t noP[5] = {0, 0, 0, 0, 0};
#define SCAN(C, ORD, U, P) scan_chunks<C, ORD>(lane, code, kid, qrow, U, preq, P, total, qc, K, list, n_pass, n_union)
            if (total > 128u) {
                if (total > 192u)
                    SCAN(4, true, 0, noP);
                else
                    SCAN(3, true, 0, noP);
            } else if (total > 64u) {
                SCAN(2, true, 0, noP);
            } else if (total != 0u) {
                SCAN(1, true, 0, noP);
            }
            // Further chunks, two or one at a time as the list has room; a full
            // list is brought down to its k smallest, and only smaller keys
            // follow.  Fewer than k: all chunks again with a wider threshold,
            // then with none but the limit.
            if (total > 256u || n_pass > (uint32_t)kPassCap || (n_pass < (uint32_t)prm.k && K != tauK)) {
                const int nch = (int)((total + 63u) >> 6);
                int u0 = 4;
                bool again = false;
                for (;;) {
#pragma unroll 1
                    for (;;) {
                        if (n_pass > (uint32_t)kPassCap) {
                            shorten_list<kListKeys / 64>(list, n_pass, K, (uint32_t)prm.k, lane, hG);
                            hK = min(tauK, max(hK, (5u << 16) | 0xFFFFu) - 0x10000u);
                        }
                        if (u0 >= nch) break;
                        const bool two = nch - u0 >= 2 && n_pass <= (uint32_t)kListKeys - 128u;
                        if (u0 + 2 <= NC) {
                            if (two)
                                SCAN(2, true, u0, noP);
                            else
                                SCAN(1, true, u0, noP);
                        } else {
                            uint32_t P[5];
                            run_starts(P, v_P, qi);
                            if (two)
                                SCAN(2, false, u0, P);
                            else
                                SCAN(1, false, u0, P);
                        }
                        u0 += two ? 2 : 1;
                    }
                    if (n_pass >= (uint32_t)prm.k || K == tauK) break;
                    K = again ? tauK : min(tauK, K + (6u << 16));
                    if (!again) hK = K;
                    again = true;
                    n_pass = n_union = 0;
                    u0 = 0;
                }
            }
#undef SCAN
            wave_sync();
            t_union += n_union;
            const uint32_t kk = min(n_pass, (uint32_t)prm.k);
            const uint32_t at = sel_n;
            if (kk != 0) {
                if (n_pass <= 64u) {
                    select_64(list, hist, n_pass, K, kk, lane, sel, sel_n, hG);
                } else {
                    select_keys<kPassSlots>(list, n_pass, K, kk, lane, sel, sel_n, hG);
                    if (n_pass > 2u * (uint32_t)prm.k) hK = min(tauK, max(hK, (5u << 16) | 0xFFFFu) - 0x10000u);
                }
            }
            v_kept = lane == qi ? (sel_n - at) | (at << 16) : v_kept;
            wave_sync();
        }
        if (lane < nq) {
            st_ranked += v_kept & 0xFFFFu;
        }
        st_union += t_union;
        finish_tile(lane, nq, q0, Q.desc, T.desc, pr.out, v_kept, sel, s_rare);
        if (!persistent) break;
    }
    for (int d = 32; d >= 1; d >>= 1) {
        st_bucket += __shfl_xor(st_bucket, d);
        st_ranked += __shfl_xor(st_ranked, d);
    }
    if (lane == 0) s_rare.add_stats(st_bucket, st_union, st_ranked);
}

// ------------------------------------------------------------------ band form (Eq. 1-2)

// Run words per query in LDS: the first place of table t's run (t stride + b_t),
// its length, then the epipolar line's three binary64 coefficients.
constexpr int kBandWords = 12 + 6;
// Places of the candidates inside the band held in LDS; more take the full scan.
constexpr int kBandCap = kPassCap;  // (so they need no bound)

// The band form: keypoints of all six runs first, the few candidates inside the
// band (about 1%) read in full and kept, or ranked as in the plain form when
// there are more than k.  Bound by L1 accesses (164 per query, 0.91 of one per
// cycle) and vector issue together: 500 x 12000 points in a band of 4 px 64 ms.
// Wide bands, 20 x 12000 points: 150 px 1.39 ms, 400 px 2.14, all 2.29 (1.88,
// 2.58 and 3.67 with the candidates in registers or a list of all of them).
__global__ __launch_bounds__(256, match_blocks_per_cu(true, 4)) void band_match_kernel(const ImgDev* __restrict__ imgs,
                                                            const PairDev* __restrict__ pairs,
                                                            const Item* __restrict__ items, int32_t n_items,
                                                            uint32_t* __restrict__ ctl, MatchParams prm,
                                                            int32_t* __restrict__ o_idx, int32_t* __restrict__ o_d1,
                                                            int32_t* __restrict__ o_d2) {
    __shared__ __attribute__((aligned(16))) uint32_t s_place[kWavesPerBlock][kBandCap];
    __shared__ __attribute__((aligned(16))) uint32_t s_list[kWavesPerBlock][kListKeys + 64];
    __shared__ __attribute__((aligned(16))) uint16_t s_sel[kWavesPerBlock][kSelCap];
    __shared__ __attribute__((aligned(16))) uint32_t s_qtab[kWavesPerBlock][kMaxTile * kBandWords];
    __shared__ Rare s_rare;
    if (threadIdx.x == 0) s_rare.fill(prm, ctl, o_idx, o_d1, o_d2);
    __syncthreads();
    const bool persistent = prm.grab > 0;
    const int lane = threadIdx.x & 63;
    const int wv = (int)uniform(threadIdx.x >> 6);
    uint32_t* place = s_place[wv];
    uint32_t* list = s_list[wv];
    uint32_t* hist = list + kListKeys;
    uint16_t* sel = s_sel[wv];
    uint32_t* qtab = s_qtab[wv];
    hist[lane] = 0u;
    uint64_t st_bucket = 0, st_ranked = 0;  // per lane
    uint64_t st_union = 0;                   // uniform
    const uint32_t tauK = ((uint32_t)prm.tau << 16) | 0xFFFFu;
    const double dd = prm.max_px * prm.max_px;
    int32_t hG = 52;  // the last ranked query's H*

    Grab grab;
    int32_t it = (int32_t)(blockIdx.x * kWavesPerBlock + wv);
    for (;;) {
        if (persistent && !grab.next(s_rare, lane, it)) break;
        if (it >= n_items) break;
        const Item item = items[it];
        const PairDev& pr = pairs[item.pair];
        const ImgDev Q = imgs[pr.qi];
        const ImgDev T = imgs[pr.ti];
        const char* code = reinterpret_cast<const char*>(T.ent);
        const char* kid = code + (size_t)kTables * T.n * 16;
        const char* kps = code + (size_t)kTables * T.n * 24;
        const int nq = (int)uniform((uint32_t)item.nq);
        const int32_t q0 = (int32_t)uniform((uint32_t)item.q0);

        // ---- setup, one lane per query of the tile
        uint32_t v_qlo, v_q4;
        uint4 v_code;
        {
            const int64_t lq = q0 + min(lane, nq - 1);
            const uint2 c0 = gload(reinterpret_cast<const uint2*>(Q.codes + 2 * lq));
            const uint2 c1 = gload(reinterpret_cast<const uint2*>(Q.codes + 2 * lq + 1));
            v_code = make_uint4(c0.x, c0.y, c1.x, c1.y);
            const uint16_t* kq = reinterpret_cast<const uint16_t*>(Q.keys + 6 * lq);
            const uint32_t k01 = gload(kq), k23 = gload(kq + 1), k45 = gload(kq + 2);
            v_qlo = k01 | (k23 << 16);
            v_q4 = k45 & 0xFFu;
            uint32_t b[kTables], e[kTables];
#pragma unroll
            for (int t = 0; t < kTables; ++t) {
                const uint32_t v = ((t < 4 ? v_qlo >> (8 * t) : k45 >> (8 * (t - 4)))) & 0xFFu;
                b[t] = gload(T.off + t * kOffStride + v);
                e[t] = gload(T.off + t * kOffStride + v + 1);
            }
            const double x = (double)gload(Q.kp + 2 * lq), y = (double)gload(Q.kp + 2 * lq + 1);
            const double la = (pr.F[0] * x + pr.F[1] * y) + pr.F[2];
            const double lb = (pr.F[3] * x + pr.F[4] * y) + pr.F[5];
            const double lc = (pr.F[6] * x + pr.F[7] * y) + pr.F[8];
            uint32_t* qt = qtab + kBandWords * lane;
            const bool own = lane < kMaxTile;
            uint32_t entries = 0;
#pragma unroll
            for (int t = 0; t < kTables; ++t) {
                const uint32_t len = e[t] - b[t];
                if (own)
                    *reinterpret_cast<uint2*>(qt + 2 * t) = make_uint2((uint32_t)t * (uint32_t)T.n + b[t], len);
                entries += len;
            }
            if (own) {
                double* ql = reinterpret_cast<double*>(qt + 12);
                ql[0] = la;
                ql[1] = lb;
                ql[2] = lc;
            }
            if (lane < nq) st_bucket += entries;
            wave_sync();
        }
        uint32_t sel_n = 0, t_union = 0;
        uint32_t v_kept = 0;  // lane qi: its kept count and first place in sel

        for (int qi = 0; qi < nq; ++qi) {
            const uint32_t* qrow = qtab + kBandWords * qi;
            uint32_t rb[kTables], rl[kTables];  // run start and length, uniform
#pragma unroll
            for (int t = 0; t < kTables; ++t) {
                const uint2 v = *reinterpret_cast<const uint2*>(qrow + 2 * t);
                rb[t] = uniform(v.x);
                rl[t] = uniform(v.y);
            }
            const double* ql = reinterpret_cast<const double*>(qrow + 12);
            const double la = ql[0], lb = ql[1], lc = ql[2];
            // band first: only keypoints are read for every bucket entry; the
            // ~1% inside the band are compacted (table, place) into LDS and
            // only they are read in full.  The runs are walked one by one, so
            // a run's table is known and its entries are consecutive: first
            // the leading 64 entries of all six with their keypoint loads in
            // flight together, then the rest of any longer run.
            // Eq. 1-2 for 64 keypoints at once: the compare's lane mask itself
            // (no branch), ANDed with the run's lanes.  Lanes past the run
            // read the entries after it: at most 64 past the keypoints of the
            // last table, inside the 512 bytes kept after the tables.
            const double rhs = dd * (la * la + lb * lb);
            auto kp_at = [&](uint32_t pos) { return gload(reinterpret_cast<const float2*>(kps + (pos << 3))); };
            auto in_band = [&](float2 kp) {
                const double xp = (double)kp.x, yp = (double)kp.y;
                const double ev = (la * xp + lb * yp) + lc;
                return ev * ev <= rhs;
            };
            uint32_t n_surv = 0;
            auto band_chunk = [&](int t, uint32_t i0, float2 kp, uint32_t pos) {
                const bool in = in_band(kp);
                const bool in_run = i0 + (uint32_t)lane < rl[t];
                const uint64_t mk = __builtin_amdgcn_ballot_w64(in) & __builtin_amdgcn_ballot_w64(in_run);
                if (mk != 0) {  // wave-uniform; most chunks have no survivor
                    const uint32_t sl = n_surv + mbcnt64(mk);
                    // a lane's own survival from its compares, not from its
                    // bit of mk (no 64-bit shift and test per lane)
                    if (in && in_run && sl < (uint32_t)kBandCap) place[sl] = ((8u * (uint32_t)t) << 24) | pos;
                    n_surv += (uint32_t)__popcll(mk);
                }
            };
            {
                uint32_t ps[kTables];
                float2 kp[kTables];
#pragma unroll
                for (int t = 0; t < kTables; ++t) ps[t] = rb[t] + (uint32_t)lane;
#pragma unroll
                for (int t = 0; t < kTables; ++t) kp[t] = kp_at(ps[t]);
#pragma unroll
                for (int t = 0; t < kTables; ++t) band_chunk(t, 0u, kp[t], ps[t]);
            }
#pragma unroll
            for (int t = 0; t < kTables; ++t) {
                for (uint32_t i0 = 64; i0 < rl[t]; i0 += 64) {
                    const uint32_t pos = rb[t] + i0 + (uint32_t)lane;
                    band_chunk(t, i0, kp_at(pos), pos);
                }
            }
            wave_sync();
            if (n_surv == 0) continue;  // v_kept stays 0

            const uint32_t qc[4] = {readlane(v_code.x, qi), readlane(v_code.y, qi), readlane(v_code.z, qi),
                                    readlane(v_code.w, qi)};
            const uint32_t qlo = readlane(v_qlo, qi), q4 = readlane(v_q4, qi);
            // the key of the entry at `pos` of table t (t8 = 8t) and, of the
            // lanes in `live`, those whose candidate counts
            auto entry = [&](uint32_t t8, uint32_t pos, uint64_t live, uint32_t& key) -> uint64_t {
                const ulonglong2 cd = gload(reinterpret_cast<const ulonglong2*>(code + (pos << 4)));
                const uint2 kw = gload(reinterpret_cast<const uint2*>(kid + (pos << 3)));
                uint32_t h = bcnt((uint32_t)cd.x ^ qc[0]);
                h = bcnt_acc((uint32_t)(cd.x >> 32) ^ qc[1], h);
                h = bcnt_acc((uint32_t)cd.y ^ qc[2], h);
                h = bcnt_acc((uint32_t)(cd.y >> 32) ^ qc[3], h);
                key = __builtin_amdgcn_alignbyte(h, kw.y, 2);
                return first_seen(kw, qlo | (uint32_t)(0xFFFFFFFFull << t8), q4) & live;
            };
            uint32_t n_pass = 0, n_union = 0, K = tauK;
            if (n_surv <= 64u) {
                const uint64_t live = ~0ull >> (64u - n_surv);
                const uint32_t e = (uint32_t)lane < n_surv ? place[lane] : 0u;
                uint32_t key;
                const uint64_t ok = entry(e >> 24, e & 0xFFFFFFu, live, key);
                n_union = (uint32_t)__popcll(ok);
                const uint64_t m = ok & __builtin_amdgcn_ballot_w64(key <= tauK);
                n_pass = (uint32_t)__popcll(m);
                if (n_pass <= (uint32_t)prm.k) {
                    // every candidate is kept: no ranking
                    if (__builtin_amdgcn_inverse_ballot_w64(m)) list_at(sel, sel_n, m) = (uint16_t)key;
                } else if (__builtin_amdgcn_inverse_ballot_w64(m)) {
                    list_at(list, 0u, m) = key;
                }
            } else {
                auto add = [&](uint64_t ok, uint32_t key) {
                    n_union += (uint32_t)__popcll(ok);
                    const uint64_t m = ok & __builtin_amdgcn_ballot_w64(key <= K);
                    if (__builtin_amdgcn_inverse_ballot_w64(m)) list_at(list, n_pass, m) = key;
                    n_pass += (uint32_t)__popcll(m);
                };
                if (n_surv <= (uint32_t)kBandCap) {
                    for (uint32_t base = 0; base < n_surv; base += 64) {
                        const uint32_t i = base + (uint32_t)lane;
                        const uint32_t e = i < n_surv ? place[i] : 0u;
                        uint32_t key;
                        const uint64_t ok = entry(e >> 24, e & 0xFFFFFFu, __builtin_amdgcn_ballot_w64(i < n_surv), key);
                        add(ok, key);
                    }
                } else {
                    // more inside the band than the places held: every entry
                    // is tested and read again, once: a list that gets full is
                    // brought down to its k smallest, and only smaller keys
                    // follow
#pragma unroll 1
                    for (int t = 0; t < kTables; ++t) {
                        const uint2 run = *reinterpret_cast<const uint2*>(qrow + 2 * t);
                        const uint32_t b = uniform(run.x), n = uniform(run.y);
#pragma unroll 1
                        for (uint32_t i0 = 0; i0 < n; i0 += 64) {
                            const uint32_t pos = b + i0 + (uint32_t)lane;
                            const uint64_t live = __builtin_amdgcn_ballot_w64(in_band(kp_at(pos))) &
                                                  __builtin_amdgcn_ballot_w64(i0 + (uint32_t)lane < n);
                            uint32_t key;
                            const uint64_t ok = entry(8u * (uint32_t)t, pos, live, key);
                            add(ok, key);
                            if (n_pass > (uint32_t)kPassCap - 64u)
                                shorten_list<kPassSlots>(list, n_pass, K, (uint32_t)prm.k, lane, hG);
                        }
                    }
                }
            }
            wave_sync();
            t_union += n_union;
            const uint32_t kk = min(n_pass, (uint32_t)prm.k);
            const uint32_t at = sel_n;
            if (n_surv <= 64u && n_pass <= (uint32_t)prm.k)
                sel_n += n_pass;  // in sel already
            else if (kk != 0 && n_pass <= 64u)
                select_64(list, hist, n_pass, K, kk, lane, sel, sel_n, hG);
            else if (kk != 0)
                select_keys<kPassSlots>(list, n_pass, K, kk, lane, sel, sel_n, hG);
            v_kept = lane == qi ? (sel_n - at) | (at << 16) : v_kept;
            wave_sync();
        }
        if (lane < nq) st_ranked += v_kept & 0xFFFFu;
        st_union += t_union;
        finish_tile(lane, nq, q0, Q.desc, T.desc, pr.out, v_kept, sel, s_rare);
        if (!persistent) break;
    }
    for (int d = 32; d >= 1; d >>= 1) {
        st_bucket += __shfl_xor(st_bucket, d);
        st_ranked += __shfl_xor(st_ranked, d);
    }
    if (lane == 0) s_rare.add_stats(st_bucket, st_union, st_ranked);
}

// ------------------------------------------------------------------ launcher
using MatchKernel = void (*)(const ImgDev*, const PairDev*, const Item*, int32_t, uint32_t*, MatchParams, int32_t*,
                             int32_t*, int32_t*);
static MatchKernel match_kernel(bool epi, int ns) {
    return epi ? band_match_kernel : ns > 4 ? plain_match_kernel<8> : plain_match_kernel<4>;
}

hipError_t launch_match(hipStream_t s, const MatchLaunch& L) {
    if (L.n_items <= 0 || L.grid <= 0) return hipSuccess;
    CH_LAUNCH(match_kernel(L.epi, L.ns), dim3((unsigned)L.grid), dim3(64 * kWavesPerBlock), 0, s, L.imgs, L.pairs,
              L.items, L.n_items, L.ctl, L.prm, L.o_idx, L.o_d1, L.o_d2);
    return hipSuccess;
}

hipError_t add_match_node(hipGraph_t graph, hipGraphNode_t* node, const hipGraphNode_t* after, const MatchLaunch& L) {
    MatchLaunch a = L;  // (the node copies the arguments)
    void* args[] = {&a.imgs, &a.pairs, &a.items, &a.n_items, &a.ctl, &a.prm, &a.o_idx, &a.o_d1, &a.o_d2};
    hipKernelNodeParams p{};
    p.func = reinterpret_cast<void*>(match_kernel(L.epi, L.ns));
    p.gridDim = dim3((unsigned)L.grid);
    p.blockDim = dim3(64 * kWavesPerBlock);
    p.kernelParams = args;
    return hipGraphAddKernelNode(node, graph, after, after ? 1 : 0, &p);
}

}  // namespace cashash
