// Pose retrieval over the history bank (Sec. 4.2, Eq. retrieval).
//
// One workgroup per query, one wave for every 256 bank entries up to 16. Each
// lane streams its share of the poses, evaluates the gates and the score in
// double precision and keeps its kLane best (score, j) pairs sorted in
// registers, together with the best pair it had to drop. The gates leave few
// candidates (a loop passes a place a few times), so the workgroup collects
// the lanes' pairs in LDS and each pair's rank is the number of pairs before
// it: no rounds of reductions. Only when there are many does each wave first
// reduce its lanes' lists to its k best with a butterfly argmin per
// result. Pairs before the best dropped one are certainly the first ones; if
// that is fewer than k, the bank is scanned again for the pairs after them
// (each scan settles at least kLane). Scores are computed with exactly the
// IEEE double operations of the definition, in the order written, with
// contraction disabled, so that the choice of chunks is reproducible bit for
// bit on the host.
//
// Large banks (more than kDirectMax entries) are cut into segments of
// kSegEntries, one workgroup of sixteen or eight waves per (query, segment), so
// that enough waves stream the bank to keep HBM busy; each leaves its segment's
// k best pairs in a workspace, and one workgroup per query merges those in the
// same order. The result is the same as the single scan.
//
// What bounds it: a bank of a few thousand poses is latency (one load batch,
// the gates, five barriers where one scan settles it), a large one the stream of
// its 64-byte poses.
// Measured per call on the device (a captured graph of calls), before (one wave per query scanning in
// turn, sorted lists of up to 32 pairs in registers, k butterfly rounds per
// wave and again per query) and now: 200 entries, k 4: 4.9 -> 4.3 us; 3000,
// k 4: 17.3 -> 8.6; 8000, k 32: 78 -> 11; 10^6, 4 queries, k 8: 62 -> 25;
// 113615, 9 queries, k 26: 696 -> 30; 2 10^6, 16 queries, k 32: 5500 -> 156;
// 2^23, k 4: 108 -> 93 (5.7 TB/s), and 110 -> 104 where 1% of it are in reach,
// 4 queries, k 8: 414 -> 177; 10^6 entries all in reach, k 4: 34.4 -> 30.0.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "internal.h"

#pragma clang fp contract(off)

namespace revisit {
namespace {

constexpr int kWave = 64;
constexpr int kMaxWaves = 16;                          // waves of a workgroup
constexpr int kSegWaves = kMaxWaves;                   // scanning waves per segment workgroup
constexpr int kSegWavesFull = 8;                       // the same, where the segments fill the chip
constexpr int kSegEntries = 16384;                     // bank entries per segment
constexpr int kDirectMax = 8192;                       // larger banks take the segmented path
constexpr int kUnroll = 4;                             // bank entries in flight per lane
constexpr int kLane = 4;                               // best pairs a lane keeps
constexpr int kMaxK = 32;
constexpr int kRankLanes = 8;                          // lanes that count one pair's rank
// Pairs are ranked by counting without a reduction first when that takes each
// thread at most so many comparisons per result wanted (and one more): as long as
// one result's round of the waves' reductions, 18 dependent lane exchanges, which get
// in each other's way when there are many waves. Measured equal at 2.5 to 4 in one
// wave (37 of 48 pairs, k 8: 7.1 us counted, 7.6 reduced; 45: 8.2 and 7.7), at 5 to 7 in
// four and eight, at 7 to 10 in sixteen (496 pairs, k 32: 31 and 40; k 16: 30 and 24).
__device__ __forceinline__ int rank_cost(int n_waves) { return 3 + 5 * (31 - __clz(n_waves)) / 4; }

// (s1, j1) strictly before (s2, j2): smaller score, then smaller index.
__device__ __forceinline__ bool before(double s1, int j1, double s2, int j2) {
    return s1 < s2 || (s1 == s2 && j1 < j2);
}

// A lane's kLane best (score, j) pairs, sorted; (INFINITY, INT32_MAX) = empty.
// (ds, dj) is the best of the pairs that were offered and are not in it.
struct LaneTop {
    double s[kLane];
    int j[kLane];
    double ds;
    int dj;

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < kLane; ++i) {
            s[i] = INFINITY;
            j[i] = INT32_MAX;
        }
        ds = INFINITY;
        dj = INT32_MAX;
    }
    // sorted insertion: slot i takes the new pair if it belongs exactly there,
    // or the pair above it if the new one goes higher up; kDrop: the pair that
    // is left over is noted
    template <bool kDrop>
    __device__ __forceinline__ void offer(double ns, int nj) {
        const bool in = before(ns, nj, s[kLane - 1], j[kLane - 1]);
        if constexpr (kDrop) {
            const double os = in ? s[kLane - 1] : ns;
            const int oj = in ? j[kLane - 1] : nj;
            if (before(os, oj, ds, dj)) {
                ds = os;
                dj = oj;
            }
        }
        if (!in) return;
#pragma unroll
        for (int i = kLane - 1; i >= 0; --i) {
            if (before(ns, nj, s[i], j[i])) {
                const bool here = i == 0 || before(s[i > 0 ? i - 1 : 0], j[i > 0 ? i - 1 : 0], ns, nj);
                s[i] = here ? ns : s[i > 0 ? i - 1 : 0];
                j[i] = here ? nj : j[i > 0 ? i - 1 : 0];
            }
        }
    }
    __device__ __forceinline__ void pop() {
#pragma unroll
        for (int i = 0; i < kLane - 1; ++i) {
            s[i] = s[i + 1];
            j[i] = j[i + 1];
        }
        s[kLane - 1] = INFINITY;
        j[kLane - 1] = INT32_MAX;
    }
};

// The wave's first pair of (s, j), in every lane.
__device__ __forceinline__ void wave_first(double& s, int& j) {
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
        const double os = __shfl_xor(s, off);
        const int oj = __shfl_xor(j, off);
        if (before(os, oj, s, j)) {
            s = os;
            j = oj;
        }
    }
}

template <int kWaves>
struct Shared {
    // what all waves' results come to, or all that one wave holds
    static constexpr int kPairs = kWaves > 1 ? kWaves * kMaxK : kLane * kWave;
    double s[kPairs];  // collected pairs, in any order
    int j[kPairs];
    double res_s[kMaxK];  // the first pairs of this scan
    int res_j[kMaxK];
    double drop_s[kWaves];
    int drop_j[kWaves];
    int out_j[kMaxK];  // chunk ids of the results so far
    int pairs, kept;
};

// kMany: k > kLane, so that pairs may be dropped and the scan repeated (k
// results at most kLane of a lane otherwise).
//
// The k first pairs of everything that scan(offer) offers, in order: calls
// put(r, s, j) for result r in one thread and returns the number found (the
// same in every thread). scan is called with offer(s, j), once per pass over
// the data, by every thread for its share. Every thread of the workgroup
// (whole waves, at most kWaves) calls this together.
template <bool kMany, int kWaves, class Scan, class Put>
__device__ __forceinline__ int first_k(Shared<kWaves>& sh, int k, Scan scan, Put put) {
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int n_waves = blockDim.x / kWave;
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    double after_s = -INFINITY;  // only pairs after this one are looked for
    int after_j = -1;
    int done = 0;
    for (;;) {
        LaneTop top;
        top.clear();
        if (tid == 0) sh.pairs = sh.kept = 0;
        scan([&](double s, int j) {
            if (!kMany || before(after_s, after_j, s, j)) top.template offer<kMany>(s, j);
        });
        __syncthreads();  // the counters are cleared, the last pass's results are read

        // the lanes' pairs into LDS when they are few
        uint64_t have[kLane];
        int mine = 0;
#pragma unroll
        for (int i = 0; i < kLane; ++i) {
            have[i] = __ballot(top.j[i] != INT32_MAX);
            mine += __popcll(have[i]);
        }
        // the wave's first pairs, one per round of a reduction: lane r gets the r-th
        auto wave_rounds = [&](int most, double& ws, int& wj) __attribute__((always_inline)) {
            ws = INFINITY;
            wj = INT32_MAX;
            int n = 0;
            for (; n < most; ++n) {
                double bs = top.s[0];
                int bj = top.j[0];
                wave_first(bs, bj);
                if (bj == INT32_MAX) break;
                if (top.j[0] == bj) top.pop();
                if (lane == n) {
                    ws = bs;
                    wj = bj;
                }
            }
            return n;
        };
        if constexpr (!kMany && kWaves == 1) {
            // one wave has its results from the reductions alone, at 0.41 us each; counting ranks
            // takes 0.06 us a pair, more from some thirty on (200 entries, k 1: 3.2 us, all
            // of them in reach 3.7; through LDS 3.5 and 4.4)
            const int found = min(k, mine);
            if (found == 1 || found * 512 <= mine * (64 + mine)) {
                double ws;
                int wj;
                wave_rounds(found, ws, wj);
                if (lane < found) {
                    put(lane, ws, wj);
                    sh.out_j[lane] = wj;
                }
                return found;
            }
        }
        int base = 0;
        if (lane == 0) {
            base = mine ? atomicAdd(&sh.pairs, mine) : 0;
            sh.drop_j[wave] = INT32_MAX;
        }
        base = __shfl(base, 0);
        if (kMany && __any(top.dj != INT32_MAX)) {
            wave_first(top.ds, top.dj);
            if (lane == 0) {
                sh.drop_s[wave] = top.ds;
                sh.drop_j[wave] = top.dj;
            }
        }
        __syncthreads();
        const int need = k - done;
        int m = sh.pairs;
        if (m <= Shared<kWaves>::kPairs && m * m <= (int)blockDim.x * rank_cost(n_waves) * (need + 1)) {
#pragma unroll
            for (int i = 0; i < kLane; ++i) {
                if (top.j[i] != INT32_MAX) {
                    const int at = base + __popcll(have[i] & below);
                    sh.s[at] = top.s[i];
                    sh.j[at] = top.j[i];
                }
                base += __popcll(have[i]);
            }
            __syncthreads();
        } else {
            double ws;
            int wj;
            const int n = wave_rounds(need, ws, wj);
            int at = 0;
            if (lane == 0 && n) at = atomicAdd(&sh.kept, n);
            at = __shfl(at, 0);
            if (lane < n) {
                sh.s[at + lane] = ws;
                sh.j[at + lane] = wj;
            }
            __syncthreads();
            m = sh.kept;
        }

        // a pair's rank is the number of pairs before it, counted by eight
        // lanes per pair (so that their LDS reads overlap)
        for (int c0 = 0; c0 < m; c0 += blockDim.x / kRankLanes) {
            const int c = c0 + tid / kRankLanes;
            const double s = c < m ? sh.s[c] : -INFINITY;
            const int j = c < m ? sh.j[c] : -1;
            int rank = 0;
#pragma unroll 4
            for (int i = tid % kRankLanes; i < m; i += kRankLanes) rank += before(sh.s[i], sh.j[i], s, j) ? 1 : 0;
#pragma unroll
            for (int off = 1; off < kRankLanes; off *= 2) rank += __shfl_xor(rank, off);
            if (c < m && tid % kRankLanes == 0 && rank < need) {
                sh.res_s[rank] = s;
                sh.res_j[rank] = j;
            }
        }
        __syncthreads();
        const int found = min(m, need);
        if constexpr (!kMany) {
            if (tid < found) {
                put(tid, sh.res_s[tid], sh.res_j[tid]);
                sh.out_j[tid] = sh.res_j[tid];
            }
            return found;
        }

        // the results before every dropped pair are certain
        double ds = INFINITY;
        int dj = INT32_MAX;
        if (lane < n_waves && sh.drop_j[lane] != INT32_MAX) {
            ds = sh.drop_s[lane];
            dj = sh.drop_j[lane];
        }
        if (__any(dj != INT32_MAX)) wave_first(ds, dj);
        int certain = found;
        if (dj != INT32_MAX) {
            certain = __popcll(__ballot(lane < found && before(sh.res_s[lane & (kMaxK - 1)], sh.res_j[lane & (kMaxK - 1)], ds, dj)));
        }
        if (tid < certain) {
            put(done + tid, sh.res_s[tid], sh.res_j[tid]);
            sh.out_j[done + tid] = sh.res_j[tid];
        }
        done += certain;
        if (done == k || dj == INT32_MAX) return done;
        after_s = sh.res_s[certain - 1];  // certain >= min(kLane, need) > 0
        after_j = sh.res_j[certain - 1];
        __syncthreads();
    }
}

// A query chunk: its centre (last column of c2w), viewing direction R e_z
// (third column), and the bank entries [lo, hi) that its index admits.
struct QueryPose {
    double cx, cy, cz, vx, vy, vz;
    int lo, hi;
};

__device__ __forceinline__ QueryPose query_pose(const RetrieveArgs& a, int qi) {
    const float* qm = a.query_c2w + (size_t)qi * 16;
    // j >= first_candidate and n - j >= delta
    const int64_t end = (int64_t)a.query_chunk[qi] - a.delta + 1;
    return QueryPose{qm[3], qm[7], qm[11], qm[2], qm[6], qm[10], max(a.first_candidate, 0),
                     (int)max((int64_t)0, min((int64_t)a.n_bank, end))};
}

// The part of bank entry j that retrieval reads: columns 2 (viewing
// direction) and 3 (centre) of the first three rows.
struct PoseCols {
    float2 r0, r1, r2;  // (R_i2, c_i) for i = 0, 1, 2
};

__device__ __forceinline__ PoseCols load_cols(const RetrieveArgs& a, int j) {
    const float* m = a.bank_c2w + (size_t)j * 16;
    return PoseCols{*reinterpret_cast<const float2*>(m + 2), *reinterpret_cast<const float2*>(m + 6),
                    *reinterpret_cast<const float2*>(m + 10)};
}

// Bank entries [begin, end) of the query's index range, kUnroll per lane at a
// time, waves in turn (each wave its own contiguous part: 2^23 entries 108 us
// instead of 102): all loads of a batch are issued before any is scored (an
// index past the end is clamped for the load and not scored), and admissible
// pairs are offered. Most entries are out of reach: those are told by the
// squared distance alone (a.reach2 is (tau_c E)^2 with a margin that no rounding
// of the definition's square root and quotient can bridge), and a batch with
// nothing in reach needs neither; otherwise the batch's square roots and
// quotients are evaluated together (one after the other behind a branch each
// they cost 10% where a few per cent of a bank of 2^23 are in reach).
//
// kEach: one after the other all the same, for workgroups of one wave, few of
// whose banks have entries in reach in all four (53 entries, k 1: 4.0 -> 3.8 us; 130
// entries, 2210 queries, k 3: 8.1 -> 7.8).
//
// kTurned: the batches start with number `turn` of them and go round.
template <bool kTurned, bool kEach, class Offer>
__device__ __forceinline__ void scan_bank(const RetrieveArgs& a, int begin, int end, int turn, const QueryPose& qp, Offer& offer) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int step = (blockDim.x / kWave) * kUnroll * kWave;
    const int64_t first = (int64_t)begin + wave * kUnroll * kWave;
    int64_t w0 = first;
    int left = 0;
    if constexpr (kTurned) {
        left = first < end ? (int)((end - first + step - 1) / step) : 0;
        if (left > 0) w0 += (int64_t)(turn % left) * step;
    }
    for (; kTurned ? left > 0 : w0 < end; w0 += step) {
        if constexpr (kTurned) {
            --left;
            if (w0 >= end) w0 = first;
        }
        const int j0 = (int)w0 + lane;  // at most 2^30 + 63
        PoseCols m[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) m[u] = load_cols(a, min(j0 + u * kWave, end - 1));
        double x[kUnroll], al[kUnroll];  // squared distance, cosine
        bool near[kUnroll], any = false;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const double dx = (double)m[u].r0.y - qp.cx;
            const double dy = (double)m[u].r1.y - qp.cy;
            const double dz = (double)m[u].r2.y - qp.cz;
            x[u] = dx * dx + dy * dy + dz * dz;
            al[u] = (double)m[u].r0.x * qp.vx + (double)m[u].r1.x * qp.vy + (double)m[u].r2.x * qp.vz;
            near[u] = j0 + u * kWave < end && !(x[u] > a.reach2) && al[u] >= a.cos_tau_v;
            any = any || near[u];
        }
        if (!__any(any)) continue;
        auto score = [&](int u, double& s) {
            const double d = sqrt(x[u]) / a.E;
            s = d + a.w_v * (1.0 - al[u]);
            near[u] = near[u] && d <= a.tau_c;
        };
        if constexpr (kEach) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (!__any(near[u])) continue;
                double s;
                score(u, s);
                if (near[u]) offer(s, j0 + u * kWave);
            }
        } else {
            double s[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) score(u, s[u]);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (near[u]) offer(s[u], j0 + u * kWave);
            }
        }
    }
}

// Result r of query qi.
__device__ __forceinline__ void put_result(const RetrieveArgs& a, int qi, int r, double s, int j) {
    a.out_idx[(size_t)qi * a.k + r] = j;
    if (a.out_score) a.out_score[(size_t)qi * a.k + r] = (float)s;
}

// What follows the results of query qi: the empty places, the count and the frame selection.
template <int kWaves>
__device__ __forceinline__ void finish(const RetrieveArgs& a, Shared<kWaves>& sh, int qi, int count) {
    const int tid = threadIdx.x;
    if (tid >= count && tid < a.k) {
        a.out_idx[(size_t)qi * a.k + tid] = -1;
        if (a.out_score) a.out_score[(size_t)qi * a.k + tid] = INFINITY;
    }
    if (tid == 0) a.out_count[qi] = count;
    if (a.out_frame_sel || a.with_slots) __syncthreads();  // out_j
    if (a.with_slots) write_stream_slots(a.slots, count, count > 0 ? sh.out_j[0] : -1, tid, blockDim.x);
    if (a.out_frame_sel) {
        const int F = a.frames_per_chunk;
        const int total = a.k * F;
        for (int t = tid; t < total; t += blockDim.x)
            a.out_frame_sel[(size_t)qi * total + t] = t / F < count ? sh.out_j[t / F] * F + (t % F) : -1;
    }
}

// The whole bank for query blockIdx.x.
template <bool kMany, int kWaves>
__global__ __launch_bounds__(kWaves * kWave) void retrieve_kernel(RetrieveArgs a) {
    __shared__ Shared<kWaves> sh;
    const int qi = blockIdx.x;
    const QueryPose qp = query_pose(a, qi);
    const int count = first_k<kMany, kWaves>(
        sh, a.k, [&](auto offer) { scan_bank<false, kWaves == 1>(a, qp.lo, qp.hi, 0, qp, offer); },
        [&](int r, double s, int j) { put_result(a, qi, r, s, j); });
    finish(a, sh, qi, count);
}

// One segment of the bank for one query: its k best pairs go to seg_s /
// seg_j [qi][seg][0 .. k), (INFINITY, INT32_MAX) past the admissible ones. The
// queries of one segment are neighbours on one XCD, so its L2 serves the bank
// to all but the first.
// 128 registers at most, four waves per SIMD: one workgroup of sixteen waves
// per compute unit, or two of eight.
template <bool kMany, int kWaves>
__global__ __launch_bounds__(kWaves * kWave, 4) void retrieve_segment_kernel(RetrieveArgs a) {
    __shared__ Shared<kWaves> sh;
    const unsigned n_items = (unsigned)a.n_seg * (unsigned)a.n_query;
    const unsigned block = row_block();
    const unsigned item = xcd_item(block, n_items);
    if (block >= xcd_grid(n_items) || item >= n_items) return;  // grid padding (uniform, before any barrier)
    const int seg = (int)(item / (unsigned)a.n_query);
    const int qi = (int)(item - (unsigned)seg * (unsigned)a.n_query);
    const QueryPose qp = query_pose(a, qi);
    const int64_t j0 = (int64_t)seg * kSegEntries;
    const int begin = (int)max(j0, (int64_t)qp.lo), end = (int)min(j0 + kSegEntries, (int64_t)qp.hi);
    const size_t base = ((size_t)qi * a.n_seg + seg) * a.k;
    auto put = [&](int r, double s, int j) {
        a.seg_s[base + r] = s;
        a.seg_j[base + r] = j;
    };
    // Two workgroups of a compute unit start together and keep in step: each at another of its
    // segment's batches, so that their loads are not all at one offset of a whole MiB
    // (2^23 entries, k 1, none in reach 100.2 -> 91.9 us, k 4, 1% in reach 110.5 -> 103.6;
    // 6 10^6 72.0 -> 72.9; sixteen waves, one workgroup after the other, have no such step).
    const int count = first_k<kMany, kWaves>(
        sh, a.k, [&](auto offer) { scan_bank<kWaves == kSegWavesFull, false>(a, begin, end, 3 * seg + (seg >> 3), qp, offer); }, put);
    if ((int)threadIdx.x >= count && (int)threadIdx.x < a.k) put(threadIdx.x, INFINITY, INT32_MAX);
}

// The results of query blockIdx.x from its n_seg * k segment results.
template <bool kMany>
__global__ __launch_bounds__(kMaxWaves * kWave) void retrieve_merge_kernel(RetrieveArgs a) {
    __shared__ Shared<kMaxWaves> sh;
    const int qi = blockIdx.x;
    const size_t base = (size_t)qi * a.n_seg * a.k;
    const int n_cand = a.n_seg * a.k;
    const int count = first_k<kMany, kMaxWaves>(
        sh, a.k,
        [&](auto offer) {
            for (int c = threadIdx.x; c < n_cand; c += blockDim.x) {
                const int j = a.seg_j[base + c];
                if (j != INT32_MAX) offer(a.seg_s[base + c], j);
            }
        },
        [&](int r, double s, int j) { put_result(a, qi, r, s, j); });
    finish(a, sh, qi, count);
}

// Waves of a workgroup over n entries, `each` per wave, as far as n_query
// workgroups do not fill the chip by themselves: past that the meeting of a
// query's waves only costs (3000 entries, 4096 queries, k 1: 67 us in twelve waves
// each, 39 in one; k 32 with every entry in reach 689 against 70; at 1024
// queries 20 in twelve, 14 in four). One wave each is also what the largest
// launches hold, 2^32 threads (the runtime takes a larger count modulo 2^32).
constexpr int kFillWaves = 4096;
dim3 waves_for(int64_t n, int each, int32_t n_query) {
    const int64_t most = kFillWaves / n_query;
    int64_t w = (n + each - 1) / each;
    w = w < kMaxWaves ? w : kMaxWaves;
    w = w < most ? w : most;
    return dim3((unsigned)(kWave * (w < 1 ? 1 : w)));
}

}  // namespace

int32_t retrieve_segments(int32_t n_bank) {
    return n_bank > kDirectMax ? (n_bank + kSegEntries - 1) / kSegEntries : 0;
}

size_t retrieve_workspace_bytes(int32_t n_bank, int32_t n_query, int32_t k) {
    const int32_t n_seg = retrieve_segments(n_bank);
    return (size_t)n_seg * n_query * k * (sizeof(double) + sizeof(int32_t));
}

template <bool kMany>
static hipError_t launch_many(const RetrieveArgs& a, hipStream_t stream) {
    if (a.n_seg == 0) {
        // one batch of loads per lane where 16 waves suffice for that: 3000 entries took 17 us in one wave, 8.8 us in twelve
        const dim3 block = waves_for(a.n_bank, kUnroll * kWave, a.n_query);
        if (block.x == kWave) hipLaunchKernelGGL((retrieve_kernel<kMany, 1>), dim3(a.n_query), block, 0, stream, a);
        else hipLaunchKernelGGL((retrieve_kernel<kMany, kMaxWaves>), dim3(a.n_query), block, 0, stream, a);
        return hipGetLastError();
    }
    const unsigned n_items = (unsigned)a.n_query * (unsigned)a.n_seg;
    // Sixteen waves of one workgroup meet with the compute unit's memory idle; past one
    // workgroup per compute unit two of eight cover each other (2^23 entries, k 4, 1% in reach
    // 113.0 -> 103.6 us, k 8, half in reach 135 -> 114.5, 4 queries 303 -> 192), which one of
    // eight does as well from half the compute units on for one query of up to kLane results
    // (2.2 10^6 entries, k 4, 1% in reach 34.7 -> 32.2; 1.5 10^6, k 1, half in reach 27.1 -> 27.9;
    // k 32, 1% in reach of 2.2 10^6 87 -> 89, of 4.2 10^6 109 -> 112; several queries read the
    // bank from the L2: 67000, 33 queries, k 3, all in reach 27.0 -> 28.4).
    if (n_items <= kFillWaves / kSegWaves / (!kMany && a.n_query == 1 ? 2 : 1))
        hipLaunchKernelGGL((retrieve_segment_kernel<kMany, kSegWaves>), dim3(xcd_grid(n_items)), dim3(kSegWaves * kWave), 0, stream, a);
    else
        hipLaunchKernelGGL((retrieve_segment_kernel<kMany, kSegWavesFull>), grid_rows(xcd_grid(n_items)), dim3(kSegWavesFull * kWave),
                           0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(retrieve_merge_kernel<kMany>, dim3(a.n_query), waves_for((int64_t)a.n_seg * a.k, kWave, a.n_query), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_retrieve(const RetrieveArgs& a, hipStream_t stream) {
    if (a.n_query == 0) return hipSuccess;
    return a.k > kLane ? launch_many<true>(a, stream) : launch_many<false>(a, stream);
}

}  // namespace revisit
