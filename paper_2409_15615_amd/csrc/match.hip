// Mutual nearest-neighbour matching of descriptor rows (reciprocity test,
// Section III-C) on gfx950 matrix cores, with exact FP64 decisions, for every
// pair of a batch at once.
//
// Sets.  Descriptor sets 2i and 2i+1 form pair i; each set is matched against
// its partner.  Set sizes live on the device; a planner lays out row slots,
// query groups and tiles.
//
// Candidates.  D(i, j) is the squared distance of two rows.  Every pair of
// sets gets a centre c and a scale s; a row x becomes the integer vector
// q = rint((x - c) / s) with |q| below 2^15 in norm, and what rounding left,
// e = ||x - c - s q|| / s, is kept with it.  The squared distance Dq of two
// integer vectors is exact in 32 bits: q = 256 h + l in signed bytes, and one
// 16x16 tile of q.q' takes four v_mfma_i32_16x16x64_i8 (h.h', h.l' + l.h',
// l.l'; 32 bits hold every sum).  By the triangle inequality the true distance
// lies within s (e + e') of s sqrt(Dq), so an upper bound of a query's second
// nearest distance becomes a threshold on Dq that no row it needs exceeds:
//   1. a sample of the partner's rows (one chunk in sample_stride) gives, per
//      query, the second smallest Dq of the sample, and with it the bound;
//   2. one sweep over the rows lists the few at or below the threshold (twice
//      the stride of them, and the rows that rounding cannot tell apart);
//   3. the listed Dq tighten the bound, and the rows that remain are scored
//      with the plain FP64 sum of squared differences in dimension order.
// Rows lie in order of their norm within tiles of 1,024: a row whose norm
// differs from a query's by more than the bound is farther than it, so both
// passes skip the chunks (16 rows) outside the band that their queries reach.
// Rows whose norm leaves the range (a handful: the scale holds rows up to
// kRangeRms times the root mean square norm) take no part in the integer
// sweep: every query that such a row could reach scores them exactly, and as
// queries they, and the queries whose list overflowed, are scanned exactly.
// The result is the exact FP64 one in every case.
//
// Forms.  Both directions in full, or (large products) one-sided: the smaller
// set of a pair against the larger, then only the rows that are some query's
// nearest neighbour back.
#include <float.h>
#include <limits.h>
#include <math.h>

#include "kmg_device.h"

namespace kmg {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileRows = 16;      // rows per chunk (MFMA M)
constexpr int kTileCols = 16;      // query columns per MFMA tile (MFMA N)
constexpr int kTilesPerWave = 4;
constexpr int kGroup = kTileCols * kTilesPerWave;  // queries per group (one wavefront)
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kPlanThreads = 1024;
constexpr int kRowBytes = 128;     // packed row: 64 high bytes, 64 low bytes
constexpr int kTileBlocks = 1024;  // grid of the tile kernels: four wavefronts per SIMD
constexpr int kTileWaves = kTileBlocks * kWavesPerBlock;
constexpr int kRounds = 2;         // tiles per resident wavefront of the sweep
constexpr int kMinDepth = 4;       // chunks per tile, at least
constexpr int kMaxDepth = 128;     // and at most
constexpr int kMaxSampleSegs = 32;
constexpr int kPartRounds = 8;     // partials of the sample in flight per query
constexpr int kCentreRows = 256;   // rows sampled for a pair's centre and scale
constexpr double kRangeRms = 4.0;
constexpr float kOrdinary = 16.0f;
constexpr double kSkew = 8.0;
constexpr double kRange = 32600.0;  // largest norm of an integer row
constexpr int kLimb = 32639;        // largest |q|: 127 * 256 + 127
constexpr int kMinCap = 16;         // listed rows per query the pool always holds
constexpr int kMaxCap = 512;
constexpr int kEmitTile = 1024;     // rows per block of the mutual test
constexpr int kSortTile = 1024;     // rows ordered by norm together
constexpr int kTileChunks = kSortTile / kTileRows;
static_assert(kTileChunks == kWave, "a lane per chunk of a sort tile");
// FP32 sums of up to 64 squares and a root, for a row and for the query, twice over
constexpr float kNormSlack = 2e-5f;
constexpr int kSortBlocks = 512;    // blocks that order rows
constexpr int kRestBlocks = 1024;   // grid of score_rest
constexpr int kFbParts = 16;        // counters per set of the queries decided on more than four scores

// Set of a flattened index given non-decreasing starts (last s with start <= t).
template <class F>
__device__ __forceinline__ int find_set(int n_sets, int64_t t, F start) {
    int lo = 0, hi = n_sets - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start(mid) <= t) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ const float* set_row(const MatchSet& s, int i, int dim) {
    return s.desc + static_cast<int64_t>(s.rows ? s.rows[i] : i) * dim;
}

// Sample stride of a set of n rows: a query's list holds about twice the
// stride, the sample pass costs 1 / stride of the sweep; below 64 rows every row
// is in the sample, so that it holds two rows whenever the set does.  Every
// stride-th chunk of a sort tile is sampled, another one of four in each tile
// (a chunk holds rows of about one norm).
__host__ __device__ __forceinline__ int sample_stride(int n) { return n < 64 ? 1 : 4; }
__device__ __forceinline__ bool in_sample(int chunk, int stride) {
    return ((chunk + chunk / kTileChunks) & (stride - 1)) == 0;
}

// ------------------------------------------------------------------ plan --

// Block-wide exclusive scan of K int32 values per thread in one pass (two
// barriers): v[k] <- the sum over lower threads, tot[k] <- the block total.
template <int K>
__device__ __forceinline__ void block_scan_k(int* v, int* tot, int* smem /* K x waves */) {
    const int lane = lane_id();
    const int wave = threadIdx.x / kWave;
    constexpr int kWaves = kPlanThreads / kWave;
    int incl[K];
#pragma unroll
    for (int k = 0; k < K; ++k) incl[k] = wave_incl_scan(v[k]);
    if (lane == kWave - 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) smem[k * kWaves + wave] = incl[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int before = 0, total = 0;
        for (int w = 0; w < kWaves; ++w) {
            const int t = smem[k * kWaves + w];
            before += w < wave ? t : 0;
            total += t;
        }
        v[k] = before + incl[k] - v[k];
        tot[k] = total;
    }
    __syncthreads();
}

// Block-wide sums of K int64 values per thread in one pass.
template <int K>
__device__ __forceinline__ void block_sum64(int64_t* v, int64_t* smem /* K x waves */) {
    constexpr int kWaves = kPlanThreads / kWave;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        v[k] = wave_sum(v[k]);
        if (lane_id() == 0) smem[k * kWaves + threadIdx.x / kWave] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = 0;
#pragma unroll 4
    for (int w = 0; w < kWaves; ++w) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] += smem[k * kWaves + w];
    }
    __syncthreads();
}

__device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }

// The query side of one phase (thread c: set c with nq queries against the
// partner's n_p rows): groups, the tiles of the sample pass and of the sweep.
// A tile is (64 queries, a run of `depth` partner chunks).  The depth is the
// least one (within [kMinDepth, kMaxDepth]) whose tiles are kRounds per resident
// wavefront: not one more, since a round that only a few wavefronts have costs
// as much as a full one; and not a single round, since a run of chunks dense
// in hits costs several times another and one wavefront then ends long after
// the rest.
// The sample of a set is split in segments of whole sort tiles, in proportion to its
// partner's tiles and about one per resident wavefront over all sets, so that a few
// queries against many rows are dealt out too: with one number of segments for all
// groups, 100,000 rows were left to eight wavefronts beside 200 queries (the call
// 595 us, now 208).
// Tiles are numbered in 32 bits, a stride of the grid past the last included: sets
// for which even the deepest tiles are more (two of 12 million rows, both directions
// in full) set err_capacity, so that nothing is matched.
constexpr int64_t kMostTiles = INT32_MAX - static_cast<int64_t>(kTileWaves);
__device__ void plan_queries(int c, bool live, int nq, int n_p, SetPlan* plan, MatchCtl* ctl, DevStatus* st,
                             int* s_scan, int64_t* s_sum) {
    const int groups = (live && n_p > 0) ? ceil_div(nq, kGroup) : 0;
    const int chunks = ceil_div(n_p, kTileRows);
    const int s_tiles = max(ceil_div(chunks, kTileChunks), 1);
    int64_t all[3] = {static_cast<int64_t>(groups) * chunks, static_cast<int64_t>(groups) * s_tiles,
                      static_cast<int64_t>(groups) * ceil_div(chunks, kMaxDepth)};
    block_sum64<3>(all, s_sum);
    if (all[2] > kMostTiles) {  // uniform
        if (live) plan[c].groups = plan[c].nq = plan[c].grp_off = plan[c].s_tile_off = plan[c].tile_off = 0;
        if (c == 0) {
            ctl->groups = ctl->s_tiles = ctl->tiles = 0;
            ctl->depth = 1;
            st->err_capacity = 1;
        }
        return;
    }
    int depth = static_cast<int>(min(max(all[0] / (kRounds * kTileWaves), static_cast<int64_t>(kMinDepth)),
                                     static_cast<int64_t>(kMaxDepth)));
    for (int it = 0; it < 4 && depth < kMaxDepth; ++it) {  // uniform
        int v[1] = {groups * ceil_div(chunks, depth)}, tot[1];
        block_scan_k<1>(v, tot, s_scan);
        if (tot[0] <= kRounds * kTileWaves) break;
        const int over = static_cast<int>(static_cast<int64_t>(depth) * tot[0] / (kRounds * kTileWaves));
        depth = min(max(over, depth + 1), kMaxDepth);
    }
    // (a set has at most 2^14 sort tiles)
    const uint32_t share = static_cast<uint32_t>(s_tiles) * kTileWaves /
                           static_cast<uint32_t>(min(max(all[1], static_cast<int64_t>(1)), static_cast<int64_t>(INT32_MAX)));
    const int s_segs = max(min(static_cast<int>(share), min(s_tiles, kMaxSampleSegs)), 1);
    int v[3] = {groups, groups * s_segs, groups * ceil_div(chunks, depth)};
    int tot[3];
    block_scan_k<3>(v, tot, s_scan);
    if (live) {
        plan[c].nq = nq;
        plan[c].groups = groups;
        plan[c].grp_off = v[0];
        plan[c].s_tile_off = v[1];
        plan[c].tile_off = v[2];
        plan[c].s_segs = s_segs;
    }
    if (c == 0) {
        ctl->groups = tot[0];
        ctl->s_tiles = tot[1];
        ctl->tiles = tot[2];
        ctl->depth = depth;
    }
}

// The rows of each sort tile (1,024 rows of a set) in order of their norm about
// zero: perm, inv, the slots' norms and the chunks' norm ranges.  A chunk so holds
// rows of nearly one norm, and a query, whose nearest rows differ from it in norm
// by no more than in distance, skips most chunks.  Needs neither the centre nor
// the scale and so runs beside the plan: within the rounding it was a chain of its
// own of 35 us, here it adds 5 us to the plan's 15.  Tiles of 2,048 rows and more, or
// one order over the whole set, leave as many products or more (a LiDAR pair 16% in
// tiles of 1,024, 20% in one order; rooms 30% and 28%).  FP32 serves: the norms only
// bound, with a margin for their rounding, what may be skipped.
__device__ void order_rows(const MatchSet* sets, int n_sets, int dim, const SinglePair& single, int first, int step,
                           const MatchWs& w) {
    constexpr int kPerRound = kSortTile / 8;
    __shared__ int s_scan[2 * (kPlanThreads / kWave)];
    __shared__ int s_tile0[kPlanThreads], s_base[kPlanThreads], s_n[kPlanThreads];
    __shared__ uint32_t s_key[kSortTile];
    __shared__ float s_nu[kSortTile];
    const bool by_value = single.on != 0;
    const int t = threadIdx.x;
    const int n = t >= n_sets ? 0 : (by_value ? (t ? single.nb : single.na) : *sets[t].n);
    int v[2] = {ceil_div(n, kTileRows), ceil_div(n, kSortTile)}, tot[2];
    block_scan_k<2>(v, tot, s_scan);
    s_n[t] = n;
    s_base[t] = v[0] * kTileRows;
    s_tile0[t] = v[1];
    __syncthreads();
    const int j = t & 7;
    for (int tile = first; tile < tot[1]; tile += step) {
        const int c = find_set(n_sets, tile, [&](int s) { return static_cast<int64_t>(s_tile0[s]); });
        const int e0 = (tile - s_tile0[c]) * kSortTile, cnt = min(kSortTile, s_n[c] - e0);
        const int64_t base = s_base[c] + e0;
        const MatchSet set = by_value ? (c ? single.b : single.a) : sets[c];
        // what there is to sort (500 pairs of clouds of 200 points: the launch 92 us with 1,024, 77)
        int size = kWave;
        while (size < cnt) size <<= 1;
#pragma unroll 4
        for (int u = 0; u < (size + kPerRound - 1) / kPerRound; ++u) {
            const int r = u * kPerRound + t / 8;
            float x2 = 0.0f;
            if (r < cnt) {
                const float* x = set_row(set, e0 + r, dim);
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const float xs = 8 * d + j < dim ? x[8 * d + j] : 0.0f;
                    x2 = fmaf(xs, xs, x2);
                }
            }
#pragma unroll
            for (int d = 1; d < 8; d <<= 1) x2 += __shfl_xor(x2, d, 8);
            if (j == 0) {
                // clamping brings norms closer, if anything; NaN, in rows that take no part, is clamped too
                const float nu = sqrtf(fminf(x2, FLT_MAX));
                s_nu[r] = nu;
                // 22 bits of the norm and the row: distinct keys (~0 for the places past the set's end)
                s_key[r] = r >= cnt ? ~0u : ((__float_as_uint(nu) >> 9) << 10) | static_cast<uint32_t>(r);
            }
        }
        __syncthreads();
        // bitonic, a key per thread: partners closer than a wavefront trade through shuffles
        uint32_t key = s_key[t];
#pragma unroll 1
        for (int k = 2; k <= size; k <<= 1) {
#pragma unroll 1
            for (int d = k >> 1; d > 0; d >>= 1) {
                uint32_t o;
                if (d >= kWave) {
                    __syncthreads();
                    s_key[t] = key;
                    __syncthreads();
                    o = s_key[t ^ d];
                } else {
                    o = __shfl_xor(key, d, kWave);
                }
                key = ((t & d) == 0) == ((t & k) == 0) ? min(key, o) : max(key, o);
            }
        }
        if (t < cnt) {
            const int row = static_cast<int>(key & 1023u);
            const int64_t slot = base + t;
            w.perm[slot] = e0 + row;
            w.inv[base + row] = e0 + t;
            w.nu[slot] = s_nu[row];
            // the chunk's norms, by the first and last row's key
            const uint32_t edge = key >> 10 << 9;
            if (t % kTileRows == 0) w.c_norm[slot / kTileRows].x = __uint_as_float(edge) * (1.0f - kNormSlack);
            if (t % kTileRows == kTileRows - 1 || t == cnt - 1)
                w.c_norm[slot / kTileRows].y = __uint_as_float(edge + 512u) * (1.0f + kNormSlack);
        }
        __syncthreads();  // the tables are free for the next tile
    }
}

// Of the 16 rows that a wavefront holds (lane d: dimension d), those with norms of at
// most kOrdinary times their upper quartile: bit 4 u for row u.  row: the lane's row, d / 4,
// is there.
__device__ __forceinline__ uint64_t ordinary_rows(const double* x, bool row) {
    constexpr int kPer = kWave / 4;
    const int d = lane_id();
    float n2[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) n2[u] = static_cast<float>(x[u]) * static_cast<float>(x[u]);
    // the lanes halve the rows that they go on with at each step, lane d ending with row d / 4
#pragma unroll
    for (int l = 32, n = kPer / 2; n > 0; l >>= 1, n >>= 1) {
#pragma unroll
        for (int u = 0; u < n; ++u) {
            const float give = d & l ? n2[u] : n2[u + n];
            n2[u] = (d & l ? n2[u + n] : n2[u]) + __shfl_xor(give, l, kWave);
        }
    }
    n2[0] += __shfl_xor(n2[0], 2, kWave);
    n2[0] += __shfl_xor(n2[0], 1, kWave);
    const float norm = n2[0] >= 0.0f ? sqrtf(n2[0]) : INFINITY;  // not a number: the largest of all
    // the quartile, to the twelve leading bits (rounded up)
    constexpr int kBits = 12;
    constexpr uint32_t kInf = 0x7f800000u;
    const uint32_t key = (row ? __float_as_uint(norm) : ~0u) >> (31 - kBits);
    const int rank = max(__popcll(ballot(row)) - 4, 0) * 3 / 4;  // four lanes a row
    uint32_t at = 0;
#pragma unroll
    for (int k = kBits - 1; k >= 0; --k)
        if (__popcll(ballot(key < (at | 1u << k))) <= rank) at |= 1u << k;
    const float most = kOrdinary * __uint_as_float(min((at + 1) << (31 - kBits), kInf));
    return ballot(row && norm <= most);
}

// One launch: block 0 plans, block 1 + i finds the centre and the scale of
// pair i, the rest order the rows.  With `single` the two sets come by value (and are written, with the
// output record, for the kernels that follow); the status is then cleared too.
//
// Centre: the mean of kCentreRows rows at even strides over both sets, in a
// fixed order (any centre is valid, every bound is stated for the rows as
// rounded); scale: kRangeRms root mean square norms about it span kRange.  Where the
// squares of the sixteen wavefronts' rows differ (their mean beyond kSkew times the
// least), rows of extraordinary norm have no part in either: a single one of a million
// times the norm among the 256 otherwise put all others within a few units, their lists
// overflowed and both sets were scanned exactly (13,015 x 15,401 rows: 261 us without
// such a row, 3,041 with it, now 252).  Looked for in every call, they cost 1 to 2.5 us.
__global__ __launch_bounds__(kPlanThreads) void match_plan(MatchSet* sets, int n_sets, int dim, int one_sided,
                                                           int64_t pool, SetPlan* plan, MatchCtl* ctl, PairScale* pp,
                                                           SinglePair single, MatchWs w, DevStatus* st) {
    const bool by_value = single.on != 0;
    const int n_pairs = n_sets / 2;
    if (static_cast<int>(blockIdx.x) > n_pairs) {
        order_rows(sets, n_sets, dim, single, static_cast<int>(blockIdx.x) - 1 - n_pairs,
                   static_cast<int>(gridDim.x) - 1 - n_pairs, w);
        return;
    }
    if (blockIdx.x > 0) {
        constexpr int kGroups = kPlanThreads / kMaxMatchDim;  // 16 row groups of 64 dimensions
        constexpr int kPer = kCentreRows / kGroups;
        static_assert(kMaxMatchDim == kWave, "a row per wavefront");
        __shared__ double s_part[kPlanThreads];
        __shared__ double s_sq[kGroups];
        __shared__ int s_rows[kGroups];
        const int pair = static_cast<int>(blockIdx.x) - 1;
        const MatchSet a = by_value ? single.a : sets[2 * pair];
        const MatchSet b = by_value ? single.b : sets[2 * pair + 1];
        const int na = by_value ? single.na : *a.n, nb = by_value ? single.nb : *b.n;
        const int64_t nt = static_cast<int64_t>(na) + nb;
        const int ns = static_cast<int>(nt < kCentreRows ? nt : kCentreRows);
        const int d = threadIdx.x % kMaxMatchDim, g = threadIdx.x / kMaxMatchDim;
        double x[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int k = g + u * kGroups;
            x[u] = 0.0;
            if (d < dim && k < ns) {
                // k nt / ns, without the division
                const int r = ns < kCentreRows ? k : static_cast<int>(static_cast<int64_t>(k) * nt / kCentreRows);
                x[u] = r < na ? set_row(a, r, dim)[d] : set_row(b, r - na, dim)[d];
            }
        }
        const bool row = g + d / 4 * kGroups < ns;
        uint64_t use = ballot(row);  // bit 4 u: row u of the wavefront counts
        double mu, all;
        int rows;
#pragma unroll 1
        for (int pass = 0;; ++pass) {
            if (d == 0) s_rows[g] = __popcll(use) / 4;
            double sum = 0.0;
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (use >> (4 * u) & 1) sum += x[u];
            s_part[threadIdx.x] = sum;
            __syncthreads();
            rows = 0;
            mu = 0.0;
            for (int q = 0; q < kGroups; ++q) {
                rows += s_rows[q];
                mu += s_part[q * kMaxMatchDim + d];
            }
            mu = rows > 0 ? mu / rows : 0.0;
            double sq = 0.0;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const double v = x[u] - mu;
                if (d < dim && (use >> (4 * u) & 1)) sq += v * v;
            }
            sq = wave_sum(sq);
            if (d == 0) s_sq[g] = sq;
            __syncthreads();
            all = 0.0;
            double least = INFINITY;
            for (int q = 0; q < kGroups; ++q) {
                all += s_sq[q];
                if (q < ns) least = fmin(least, s_sq[q]);
            }
            if (pass > 0 || all <= kSkew * kGroups * least) break;  // uniform; what is not a number goes on
            use = ordinary_rows(x, row);
        }
        if (g == 0) pp[pair].mu[d] = d < dim ? mu : 0.0;
        if (threadIdx.x == 0) {
            const double rms = rows > 0 ? sqrt(all / rows) : 0.0;
            double s = rms * (kRangeRms / kRange);
            if (!(s > 1e-30) || !(s < 1e30)) s = 1.0;  // equal rows, or nothing that can be scaled
            pp[pair].scale = s;
            pp[pair].inv = 1.0 / s;
        }
        return;
    }
    __shared__ int s_scan[3 * (kPlanThreads / kWave)];
    __shared__ int64_t s_sum[3 * (kPlanThreads / kWave)];
    const int c = threadIdx.x;
    if (by_value) {
        for (int k = c; k < static_cast<int>(sizeof(DevStatus) / 4); k += kPlanThreads)
            reinterpret_cast<uint32_t*>(st)[k] = 0u;
        if (c == 0) {
            single.counts[0] = single.na;
            single.counts[1] = single.nb;
            MatchSet a = single.a, b = single.b;
            a.n = single.counts;
            b.n = single.counts + 1;
            sets[0] = a;
            sets[1] = b;
            *single.out_dev = single.out;
        }
        __syncthreads();
    }
    const bool live = c < n_sets;
    const bool paired = live && (c ^ 1) < n_sets;
    const int n = !live ? 0 : (by_value ? (c ? single.nb : single.na) : *sets[c].n);
    const int n_p = !paired ? 0 : (by_value ? (c ? single.na : single.nb) : *sets[c ^ 1].n);
    const int chunks = ceil_div(n, kTileRows);
    const int emit = (c & 1) ? 0 : (paired ? max(1, ceil_div(n, kEmitTile)) : 0);
    int v[2] = {chunks, emit};
    int tot[2];
    block_scan_k<2>(v, tot, s_scan);
    // one buffer descriptor spans a set's packed rows: keep them below 2 GiB
    if (static_cast<int64_t>(chunks) * kTileRows * kRowBytes > INT32_MAX) st->err_capacity = 1;
    if (live) {
        SetPlan pl{};
        pl.n = n;
        pl.base = v[0] * kTileRows;
        pl.emit_off = v[1];
        plan[c] = pl;
    }
    // one-sided: the larger set of each pair (the second on a tie) brings rows only
    const bool rows_only = one_sided && ((c & 1) ? n >= n_p : n > n_p);
    const int nq = (!paired || rows_only) ? 0 : n;
    __syncthreads();
    plan_queries(c, live, nq, n_p, plan, ctl, st, s_scan, s_sum);
    if (c == 0) {
        ctl->slots = tot[0] * kTileRows;
        ctl->emit_tiles = tot[1];
        // whole 128-byte lines, an odd number of them: with lists a power of two apart the first
        // lines of all lists fall on the same memory channels
        const int64_t cap = pool / max(tot[0] * kTileRows, 1);
        const int lines = static_cast<int>((cap < kMaxCap ? cap : kMaxCap) / 16);
        ctl->cap = 16 * (lines - 1 + (lines & 1));
        ctl->open = 0;
        ctl->n_long = 0;
    }
}

// The plan of the matching back (the image rows of every set as queries).
__global__ __launch_bounds__(kPlanThreads) void match_plan_back(int n_sets, SetPlan* plan, MatchCtl* ctl,
                                                                DevStatus* st) {
    __shared__ int s_scan[3 * (kPlanThreads / kWave)];
    __shared__ int64_t s_sum[3 * (kPlanThreads / kWave)];
    const int c = threadIdx.x;
    const bool live = c < n_sets && (c ^ 1) < n_sets;
    const int n_p = live ? plan[c ^ 1].n : 0;
    const int nq = live ? plan[c].n_img : 0;
    if (live) plan[c].n_open = 0;
    plan_queries(c, live, nq, n_p, plan, ctl, st, s_scan, s_sum);
    if (c == 0) ctl->open = ctl->n_long = 0;
}

// ------------------------------------------------------------- rounding --

// What the integer sweep knows of a row: half its squared norm, negated, less
// one (kNoRow: the row takes no part, its score is below every least score),
// and how far rounding moved it (in units of the scale, rounded up).
constexpr int kNoRow = INT_MIN;
__device__ __forceinline__ int half_norm(uint32_t n2) { return -static_cast<int>(n2 >> 1) - 1; }
// Rounding moves a coordinate by at most half a unit: the error of any row.
__device__ __forceinline__ double most_err(int dim) { return 0.5 * sqrt(static_cast<double>(dim)) * (1.0 + 1e-6) + 1e-4; }

// Packed rows: chunks of 16 rows, 2 KB each, the high bytes first; piece
// (g, r) of a half holds bytes 16 g .. 16 g + 15 of row r, where lane 16 g + r
// of a tile's load finds it (a half is one contiguous 1 KB load).
__device__ __forceinline__ int64_t piece_at(int64_t row, int half, int g) {
    return (row / kTileRows) * (kTileRows * kRowBytes) + half * (kTileRows * kRowBytes / 2) +
           (g * kTileRows + row % kTileRows) * 16;
}

// Eight lanes per row (lane j: dimensions 8 j .. 8 j + 7): the row's bytes, its
// norm and rounding error, into its slot.  Also readies the slot for the passes that follow.
// Bound by the descriptors' reads and the packed rows' writes (4 dim + 160
// bytes a row).
__global__ __launch_bounds__(kBlock) void match_round(const MatchSet* __restrict__ sets, SetPlan* plan, int n_sets,
                                                      int dim, const PairScale* __restrict__ pp, MatchWs w,
                                                      const MatchCtl* __restrict__ ctl) {
    const int64_t slots = ctl->slots;
    const int64_t tid = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t gs = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t k = tid; k <= ctl->emit_tiles; k += gs) w.emit_status[k] = 0ull;
    for (int64_t k = tid; k < slots / kWave + n_sets + 1; k += gs) w.grp_done[k] = 0;
    for (int64_t k = tid; k < n_sets * kFbParts; k += gs) w.fb_part[k] = 0;
    for (int64_t k = tid; k < 2 * kMaxWorkCounters; k += gs) w.work[k] = 0;
    const int j = threadIdx.x & 7;
    for (int64_t slot = tid / 8; slot < slots; slot += gs / 8) {
        const int c = find_set(n_sets, slot, [&](int s) { return static_cast<int64_t>(plan[s].base); });
        const int at = static_cast<int>(slot) - plan[c].base;
        const bool row = at < plan[c].n;
        const int i = row ? w.perm[slot] : 0;
        const double s = pp[c >> 1].scale, inv = pp[c >> 1].inv;
        uint2 vh = make_uint2(0u, 0u), vl = make_uint2(0u, 0u);
        unsigned long long n2 = 0ull;
        double e2 = 0.0;
        bool ok = true;
        if (row) {
            const float* x = set_row(sets[c], i, dim);
            uint32_t hi[2] = {0u, 0u}, lo[2] = {0u, 0u};
            float xs[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) xs[u] = 8 * j + u < dim ? x[8 * j + u] : 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (8 * j + u >= dim) continue;
                const double v = static_cast<double>(xs[u]) - pp[c >> 1].mu[8 * j + u];
                const double t = rint(v * inv);
                const bool in = fabs(t) <= static_cast<double>(kLimb);  // false for NaN too
                ok = ok && in;
                const int q = in ? static_cast<int>(t) : 0;
                const double r = (v - static_cast<double>(q) * s) * inv;
                e2 += r * r;
                n2 += static_cast<unsigned long long>(static_cast<long long>(q) * q);
                const int l = static_cast<int>(static_cast<signed char>(q & 255));
                const int h = (q - l) >> 8;
                hi[u >> 2] |= static_cast<uint32_t>(h & 255) << (8 * (u & 3));
                lo[u >> 2] |= static_cast<uint32_t>(l & 255) << (8 * (u & 3));
            }
            vh = make_uint2(hi[0], hi[1]);
            vl = make_uint2(lo[0], lo[1]);
        }
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            n2 += __shfl_xor(n2, d, 8);
            e2 += __shfl_xor(e2, d, 8);
            ok = (__shfl_xor(ok ? 1 : 0, d, 8) != 0) && ok;
        }
        const bool out = row && !(ok && static_cast<double>(n2) <= kRange * kRange);
        if (out) vh = vl = make_uint2(0u, 0u);
        const int hn = row && !out ? half_norm(static_cast<uint32_t>(n2)) : kNoRow;
        *reinterpret_cast<uint2*>(w.rows + piece_at(slot, 0, j >> 1) + 8 * (j & 1)) = vh;
        *reinterpret_cast<uint2*>(w.rows + piece_at(slot, 1, j >> 1) + 8 * (j & 1)) = vl;
        if (j == 0) {
            w.half[slot] = hn;
            w.cnt[slot] = 0;
            if (row) w.nn[plan[c].base + i] = -1;
            // rounded up: the residuals come from a handful of FP64 roundings; < 0: not in the sweep
            w.err[slot] = row && !out ? static_cast<float>(sqrt(e2) * (1.0 + 1e-6)) + 1e-4f : -1.0f;
            if (out) w.out_list[plan[c].base + atomicAdd(&plan[c].n_out, 1)] = i;
        }
    }
}

// --------------------------------------------------------- integer tiles --

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kBufferWord3 = 0x00020000u;  // raw buffer, 32-bit data format (gfx9)

// A score stands for the squared distance: w = q.q' - floor(n / 2) - floor(n' / 2) - 1
// = -1 - Dq / 2 up to the parities dropped, so -2 (w + 1) lies in [Dq - 2, Dq]
// and a larger score is a nearer row.  Dq < 2^32 for rows within kRange.  The
// tiles work on raw scores, without the query's half norm.
__device__ __forceinline__ double score_d2(int w) { return -2.0 * (static_cast<double>(w) + 1.0); }

// The least score of a row that a query may need, given a score `w2` that two
// rows reach and the summed rounding errors e of the query and of any row:
// sqrt(Dq) <= sqrt(D2 + 2) + 2 e (see the head of this file).
__device__ __forceinline__ int least_score(int w2, double e) {
    if (w2 == kNoRow) return INT_MIN + 1;  // fewer than two rows known: every row
    const double r = sqrt(score_d2(w2) + 2.0) + 2.0 * e;
    const double t = 0.5 * r * r * (1.0 + 1e-9) + 2.0;
    return t >= 2147483646.0 ? INT_MIN + 1 : -2 - static_cast<int>(t);
}

// Rows of one set as the tiles read them: raw buffer loads keep their place
// ahead of the products (plain loads get sunk to their first use), and an
// offset past the range reads zeros.
struct RowBuf {
    __amdgpu_buffer_rsrc_t rows, half;
};
__device__ __forceinline__ RowBuf row_buf(const unsigned char* rows, const int* half, int64_t base, int chunks) {
    RowBuf b;
    b.rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(rows + base * kRowBytes), 0,
                                               chunks * kTileRows * kRowBytes, static_cast<int>(kBufferWord3));
    b.half = __builtin_amdgcn_make_buffer_rsrc(const_cast<int*>(half + base), 0, chunks * kTileRows * 4,
                                               static_cast<int>(kBufferWord3));
    return b;
}
struct ChunkRegs {
    i32x4 h, l, n;
};
// Lane: row lane % 16 of the chunk, bytes 16 (lane / 16) ..; and the half
// norms of rows 4 (lane / 16) .. + 3, the result rows the lane holds.
__device__ __forceinline__ ChunkRegs load_chunk(const RowBuf& b, int chunk, int lane) {
    const int off = chunk * (kTileRows * kRowBytes);
    ChunkRegs r;
    r.h = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(b.rows, lane * 16, off, 0));
    r.l = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(b.rows, lane * 16 + 1024, off, 0));
    r.n = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(b.half, (lane >> 4) * 16, chunk * 64, 0));
    return r;
}

// The queries of a group as the tiles hold them (lane: column lane % 16 of
// every 16-query tile); columns past the last query repeat it.
struct QueryRegs {
    i32x4 h[kTilesPerWave], l[kTilesPerWave];
    int slot[kTilesPerWave];
};
__device__ __forceinline__ QueryRegs load_queries(const SetPlan& qc, const int32_t* __restrict__ list, int g,
                                                  const unsigned char* __restrict__ rows, int lane) {
    QueryRegs q;
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) {
        const int i = min(g * kGroup + t * kTileCols + (lane & 15), qc.nq - 1);
        q.slot[t] = list ? list[qc.base + i] : qc.base + i;
    }
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) {
        q.h[t] = *reinterpret_cast<const i32x4*>(rows + piece_at(q.slot[t], 0, lane >> 4));
        q.l[t] = *reinterpret_cast<const i32x4*>(rows + piece_at(q.slot[t], 1, lane >> 4));
    }
    return q;
}

// Raw scores of a chunk's 16 rows against one 16-query tile: lane l holds
// column l % 16 and rows 4 (l / 16) + 0..3.
__device__ __forceinline__ i32x4 tile_scores(const ChunkRegs& a, const i32x4& qh, const i32x4& ql) {
    i32x4 w = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.h, qh, i32x4{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = static_cast<int>(static_cast<uint32_t>(w[r]) << 8);
    w = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.h, ql, w, 0, 0, 0);
    w = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.l, qh, w, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = static_cast<int>((static_cast<uint32_t>(w[r]) << 8) + static_cast<uint32_t>(a.n[r]));
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a.l, ql, w, 0, 0, 0);
}

// Raw scores of a chunk's 16 rows against the four 16-query tiles: lane l
// holds column l % 16 and rows 4 (l / 16) + 0..3 of each.  The partial sums go
// through the products' accumulators, shifted between them (all sums modulo
// 2^32, which hold the result): eight vector instructions a tile beside the
// 64 cycles of its four products; the tiles' chains interleave.
__device__ __forceinline__ void group_scores(const ChunkRegs& a, const QueryRegs& q, i32x4* w) {
    const i32x4 z = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) w[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.h, q.h[t], z, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) w[t][r] = static_cast<int>(static_cast<uint32_t>(w[t][r]) << 8);
        w[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.h, q.l[t], w[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) w[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.l, q.h[t], w[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            w[t][r] = static_cast<int>((static_cast<uint32_t>(w[t][r]) << 8) + static_cast<uint32_t>(a.n[r]));
        w[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.l, q.l[t], w[t], 0, 0, 0);
    }
}

// Runs use(chunk registers, chunk) over the chunks base + (set bits of todo),
// the next chunk's loads ahead of its use.  (A second chunk ahead, in a loop of
// three register sets, was no faster: the loop is bound by issue, not by the
// loads.)
template <class F>
__device__ __forceinline__ void for_chunks(const RowBuf& b, int base, uint64_t todo, int lane, F use) {
    if (!todo) return;  // uniform
    int k = base + __builtin_ctzll(todo);
    ChunkRegs next = load_chunk(b, k, lane);
    do {
        todo &= todo - 1;
        const int kn = todo ? base + __builtin_ctzll(todo) : k;
        const ChunkRegs a = next;
        next = load_chunk(b, kn, lane);
        __builtin_amdgcn_sched_barrier(0);
        use(a, k);
        __builtin_amdgcn_sched_barrier(0);
        k = kn;
    } while (todo);
}

// How far the nearest rows of a query can lie, given a score that two rows
// reach and the summed rounding errors, in the descriptors' units, rounded up.
__device__ __forceinline__ float reach_of(int w2, double e, double scale) {
    if (w2 == kNoRow) return INFINITY;
    return static_cast<float>((sqrt(score_d2(w2) + 2.0) + e) * scale * (1.0 + 1e-6) + 1e-18);  // and squares that underflow
}

__device__ __forceinline__ int med3(int a, int b, int c) { return max(min(a, b), min(max(a, b), c)); }

// First of a wavefront's tiles (every kTileWaves-th).  A batch's tiles are dealt to
// the XCDs in runs of kTileRun, which are neighbouring groups against the same
// chunks: dealt one by one each of the eight L2s loaded every pair's rows, and the
// sweep ran at the memory's rate (64 pairs 2.60 -> 2.29 ms, 16 pairs 596 -> 515 us).
// The rows of a single pair come from the last-level cache either way, and dealt
// one by one its dense runs spread more evenly (two sets of 15,000: 76 us against
// 79; whole eighths per XCD were slower still, by a tenth).
constexpr int kTileRun = 128;
static_assert(kTileWaves % (kXcds * kTileRun) == 0, "a permutation of the wavefronts");
__device__ __forceinline__ int first_tile(int n_sets, int wv) {
    const int b = static_cast<int>(blockIdx.x);
    if (n_sets <= 2) return b * kWavesPerBlock + wv;
    const int j = b / kXcds * kWavesPerBlock + wv;  // within the XCD
    return j / kTileRun * (kXcds * kTileRun) + b % kXcds * kTileRun + j % kTileRun;
}

// The 16 x 16 products that a wavefront evaluated, where they are counted (kCount: per-stage
// timing is on; counted always they were 1% of the call for 100,000 rows), into counters a
// line each (all into one, the sample pass of a LiDAR pair took 62 us instead of 36).
__device__ __forceinline__ void count_work(int64_t* work, int done) {
    constexpr int kApart = 8;
    if (done && lane_id() == 0)
        atomicAdd(reinterpret_cast<unsigned long long*>(work) + global_wave() % (kMaxWorkCounters / kApart) * kApart,
                  static_cast<unsigned long long>(done) * (kTileRows * kTileCols));
}

// Best and second best raw score of every query over a segment of the sample
// (whole sort tiles).  Of each sort tile the chunks in the group's own norm range
// go first; what they find limits the norms at which the rest can matter.
template <bool kCount>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void sample_tiles(
    const SetPlan* __restrict__ plan, int n_sets, int dim, const int32_t* __restrict__ list,
    const PairScale* __restrict__ pp, MatchWs w, const MatchCtl* __restrict__ ctl, const DevStatus* __restrict__ st,
    int64_t* work) {
    const int lane = lane_id();
    const int total = st->err_capacity ? 0 : ctl->s_tiles;
    int done = 0;  // 16 x 16 products
    for (int tile = first_tile(n_sets, static_cast<int>(threadIdx.x / kWave)); tile < total; tile += kTileWaves) {
        const int tu = __builtin_amdgcn_readfirstlane(tile);
        const int c = find_set(n_sets, tu, [&](int s) { return static_cast<int64_t>(plan[s].s_tile_off); });
        const SetPlan qc = plan[c], pc = plan[c ^ 1];
        const int chunks = ceil_div(pc.n, kTileRows), tiles = max(ceil_div(chunks, kTileChunks), 1);
        const int segs = qc.s_segs;
        const int stride = sample_stride(pc.n);
        const int local = tu - qc.s_tile_off;
        const int g = local % qc.groups, sg = local / qc.groups;
        const int t0 = static_cast<int>(static_cast<int64_t>(tiles) * sg / segs);
        const int t1 = static_cast<int>(static_cast<int64_t>(tiles) * (sg + 1) / segs);
        const RowBuf b = row_buf(w.rows, w.half, pc.base, chunks);
        const QueryRegs q = load_queries(qc, list, g, w.rows, lane);
        // the norms of the group and of each 16 queries (those out of range left out), and the
        // queries' half norms by column
        float lo[kTilesPerWave], hi[kTilesPerWave];
        int own[kTilesPerWave];
        {
            const int i = g * kGroup + lane;
            const int slot = list ? list[qc.base + min(i, qc.nq - 1)] : qc.base + min(i, qc.nq - 1);
            const bool act = i < qc.nq && w.err[slot] >= 0.0f;
            const float nu = w.nu[slot];
            const int half = w.half[slot];
            float l = act ? nu * (1.0f - kNormSlack) : INFINITY, h = act ? nu * (1.0f + kNormSlack) : -INFINITY;
#pragma unroll
            for (int d = 1; d < kTileCols; d <<= 1) {
                l = fminf(l, __shfl_xor(l, d, kWave));
                h = fmaxf(h, __shfl_xor(h, d, kWave));
            }
            const int o = act ? half + 1 : kNoRow;
#pragma unroll
            for (int t = 0; t < kTilesPerWave; ++t) {
                own[t] = __shfl(o, t * kTileCols + (lane & 15), kWave);
                lo[t] = __shfl(l, t * kTileCols, kWave);
                hi[t] = __shfl(h, t * kTileCols, kWave);
            }
        }
        const float lo_g = fminf(fminf(lo[0], lo[1]), fminf(lo[2], lo[3]));
        const float hi_g = fmaxf(fmaxf(hi[0], hi[1]), fmaxf(hi[2], hi[3]));
        const double scale = pp[c >> 1].scale;
        int m1[kTilesPerWave], m2[kTilesPerWave];
#pragma unroll
        for (int t = 0; t < kTilesPerWave; ++t) m1[t] = m2[t] = kNoRow;
        const auto see = [&](const ChunkRegs& a, int) {
            i32x4 s[kTilesPerWave];
            group_scores(a, q, s);
#pragma unroll
            for (int t = 0; t < kTilesPerWave; ++t) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    m2[t] = med3(m1[t], m2[t], s[t][r]);
                    m1[t] = max(m1[t], s[t][r]);
                }
            }
        };
        // the chunks of sort tile tl in the sample, and their norms
        const auto chunk_norms = [&](int tl, bool& have) {
            const int k = tl * kTileChunks + lane;
            have = k < chunks && in_sample(k, stride);
            return w.c_norm[pc.base / kTileRows + max(min(k, chunks - 1), 0)];
        };
        const auto near_of = [&](const float2& cn, bool have) { return ballot(have && cn.x <= hi_g && cn.y >= lo_g); };
        for (int tl = t0; tl < t1; ++tl) {
            bool have;
            const float2 cn = chunk_norms(tl, have);
            const uint64_t near = near_of(cn, have);
            if (kCount) done += kTilesPerWave * __popcll(near);
            for_chunks(b, tl * kTileChunks, near, lane, see);
        }
        for (int tl = t0; tl < t1; ++tl) {
            bool have;
            const float2 cn = chunk_norms(tl, have);
            // the farthest that a query of each 16 may have to look, by what its column knows
            uint64_t need[kTilesPerWave];
#pragma unroll
            for (int t = 0; t < kTilesPerWave; ++t) {
                int a1 = m1[t], a2 = m2[t];
#pragma unroll
                for (int d = 16; d < kWave; d <<= 1) {
                    const int o1 = __shfl_xor(a1, d, kWave), o2 = __shfl_xor(a2, d, kWave);
                    a2 = max(min(a1, o1), max(a2, o2));
                    a1 = max(a1, o1);
                }
                int least = own[t] == kNoRow ? INT_MAX : (a2 == kNoRow ? kNoRow : a2 + own[t]);
#pragma unroll
                for (int d = 1; d < kTileCols; d <<= 1) least = min(least, __shfl_xor(least, d, kWave));
                const float reach = least == INT_MAX ? 0.0f : reach_of(least, 2.0 * most_err(dim), scale);
                need[t] = ballot(have && cn.x <= hi[t] + reach && cn.y >= lo[t] - reach);
            }
            const uint64_t near = near_of(cn, have);
            const uint64_t rest = ((need[0] | need[1]) | (need[2] | need[3])) & ~near;
#pragma unroll
            for (int t = 0; t < kTilesPerWave; ++t)
                if (kCount) done += __popcll(need[t] & ~near);
            for_chunks(b, tl * kTileChunks, rest, lane, [&](const ChunkRegs& a, int k) {
#pragma unroll
                for (int t = 0; t < kTilesPerWave; ++t) {
                    if (!((need[t] >> (k - tl * kTileChunks)) & 1)) continue;  // uniform
                    const i32x4 s = tile_scores(a, q.h[t], q.l[t]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        m2[t] = med3(m1[t], m2[t], s[r]);
                        m1[t] = max(m1[t], s[r]);
                    }
                }
            });
        }
        // the four row groups of a column
#pragma unroll
        for (int t = 0; t < kTilesPerWave; ++t) {
#pragma unroll
            for (int d = 16; d < kWave; d <<= 1) {
                const int o1 = __shfl_xor(m1[t], d, kWave), o2 = __shfl_xor(m2[t], d, kWave);
                m2[t] = max(min(m1[t], o1), max(m2[t], o2));
                m1[t] = max(m1[t], o1);
            }
            if (lane < 16)
                w.s_best[static_cast<int64_t>(tu) * kGroup + t * kTileCols + lane] = make_int2(m1[t], m2[t]);
        }
    }
    if (kCount) count_work(work, done);
}

constexpr int kStage = 384;  // hits a wavefront gathers in LDS before it hands them out

// The sweep: every row at or above a query's least score goes to the query's
// list (row, raw score).  Chunks whose norms no query of a 16-query tile can
// reach are passed over, without their loads where no tile of the group needs
// them: a scan pair keeps a sixth to a quarter of the products, indoor rooms a
// quarter to two fifths (15,000 rows a side: 150 us -> 101 us; two sets of
// 100,000: 3.5 ms -> 2.0 ms).  A chunk that all four tiles need runs their products
// interleaved.  What is left is dense in hits: a lane's four scores go to LDS as
// they are (one write per lane with a hit; sorting the single hits out on the
// spot was a quarter of the time, 101 us -> 78 us) and are handed out when the
// stage is full: ranked per query in LDS, with one global atomic per query.
// Consecutive tiles sweep the same run of chunks for consecutive groups, so the
// run is read from cache; loads run a chunk ahead.  What bounds it: for rows that the
// norms cannot prune, the products; for a LiDAR pair the waits (matrix unit 16%,
// vector unit 24% busy), which loads two chunks ahead, three wavefronts per SIMD or one
// or three rounds of tiles only made longer (87 us -> 89 to 98).
template <bool kCount>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void sweep_tiles(
    const SetPlan* __restrict__ plan, int n_sets, int dim, const int32_t* __restrict__ list,
    const PairScale* __restrict__ pp, MatchWs w, const MatchCtl* __restrict__ ctl, const DevStatus* __restrict__ st,
    int64_t* work) {
    __shared__ i32x4 s_hit[kWavesPerBlock][kStage];     // a lane's four scores,
    __shared__ uint32_t s_at[kWavesPerBlock][kStage];   // their first row and column,
    __shared__ uint16_t s_rank[kWavesPerBlock][kStage]; // and the place of the first in its list
    __shared__ int s_least[kWavesPerBlock][kGroup];
    __shared__ int s_cnt[kWavesPerBlock][kGroup];
    __shared__ int s_slot[kWavesPerBlock][kGroup];
    const int lane = lane_id();
    const int wv = threadIdx.x / kWave;
    const int total = st->err_capacity ? 0 : ctl->tiles;
    const int cap = ctl->cap, depth = ctl->depth;
    const double e_rows = most_err(dim);
    int done = 0;
    for (int tile = first_tile(n_sets, wv); tile < total; tile += kTileWaves) {
        const int tu = __builtin_amdgcn_readfirstlane(tile);
        const int c = find_set(n_sets, tu, [&](int s) { return static_cast<int64_t>(plan[s].tile_off); });
        const SetPlan qc = plan[c], pc = plan[c ^ 1];
        const int chunks = ceil_div(pc.n, kTileRows);
        const int local = tu - qc.tile_off;
        const int g = local % qc.groups, sg = local / qc.groups;
        const int c0 = sg * depth, c1 = min(c0 + depth, chunks);
        const RowBuf b = row_buf(w.rows, w.half, pc.base, chunks);
        const QueryRegs q = load_queries(qc, list, g, w.rows, lane);
        // query `lane` of the group: its slot and the least raw score of a row that it may need
        // (the sample's partials, all in flight; the chain per tile column took 13 us)
        const int iq = g * kGroup + lane;
        const int slot_l = list ? list[qc.base + min(iq, qc.nq - 1)] : qc.base + min(iq, qc.nq - 1);
        const float err = w.err[slot_l];
        const int own = w.half[slot_l] + 1;  // minus the query's half norm
        const int2* src = w.s_best + static_cast<int64_t>(qc.s_tile_off + g) * kGroup + lane;
        const int64_t seg_step = static_cast<int64_t>(qc.groups) * kGroup;
        int m1 = kNoRow, m2 = kNoRow;
#pragma unroll 1
        for (int k0 = 0; k0 < qc.s_segs; k0 += kPartRounds) {
            int2 part[kPartRounds];
#pragma unroll
            for (int k = 0; k < kPartRounds; ++k) part[k] = src[min(k0 + k, qc.s_segs - 1) * seg_step];
#pragma unroll
            for (int k = 0; k < kPartRounds; ++k) {
                if (k0 + k >= qc.s_segs) break;
                m2 = max(min(m1, part[k].x), max(m2, part[k].y));
                m1 = max(m1, part[k].x);
            }
        }
        const bool act = iq < qc.nq && err >= 0.0f;
        const int w2 = m2 == kNoRow ? m2 : m2 + own;
        const double e = static_cast<double>(err) + e_rows;
        // never below the score of a row that takes no part
        const int least_l = act ? max(least_score(w2, e) - own, INT_MIN + 1) : INT_MAX;
        int least[kTilesPerWave];
#pragma unroll
        for (int t = 0; t < kTilesPerWave; ++t) least[t] = __shfl(least_l, t * kTileCols + (lane & 15), kWave);
        // the norms that each 16-query tile may need, and the chunks of the run that hold some
        const float nu = w.nu[slot_l], reach = reach_of(w2, e, pp[c >> 1].scale);
        float lo = act ? nu * (1.0f - kNormSlack) - reach : INFINITY, hi = act ? nu * (1.0f + kNormSlack) + reach : -INFINITY;
#pragma unroll
        for (int d = 1; d < kTileCols; d <<= 1) {
            lo = fminf(lo, __shfl_xor(lo, d, kWave));
            hi = fmaxf(hi, __shfl_xor(hi, d, kWave));
        }
        s_least[wv][lane] = least_l;
        s_slot[wv][lane] = slot_l;
        int n_hit = 0;
        const auto hand_out = [&]() {
            s_cnt[wv][lane] = 0;
            __builtin_amdgcn_wave_barrier();
#pragma unroll 1
            for (int k = lane; k < n_hit; k += kWave) {
                const int col = static_cast<int>(s_at[wv][k] >> 26);
                const i32x4 v = s_hit[wv][k];
                const int lt = s_least[wv][col];
                s_rank[wv][k] = static_cast<uint16_t>(
                    atomicAdd(&s_cnt[wv][col], (v[0] >= lt) + (v[1] >= lt) + (v[2] >= lt) + (v[3] >= lt)));
            }
            __builtin_amdgcn_wave_barrier();
            const int mine = s_cnt[wv][lane];
            s_cnt[wv][lane] = mine ? atomicAdd(&w.cnt[slot_l], mine) : 0;
            __builtin_amdgcn_wave_barrier();
#pragma unroll 1
            for (int k = lane; k < n_hit; k += kWave) {
                const uint32_t where = s_at[wv][k];
                const int col = static_cast<int>(where >> 26);
                const i32x4 v = s_hit[wv][k];
                const int lt = s_least[wv][col];
                int at = s_cnt[wv][col] + s_rank[wv][k];
                uint2* out = w.pool + static_cast<int64_t>(s_slot[wv][col]) * cap;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (v[r] < lt) continue;
                    if (at < cap) out[at] = make_uint2((where & 0x3ffffffu) + r, static_cast<uint32_t>(v[r]));
                    ++at;
                }
            }
            __builtin_amdgcn_wave_barrier();
            n_hit = 0;
        };
        for (int k0 = c0; k0 < c1; k0 += kWave) {
            // the chunks that each 16 queries need
            uint64_t need[kTilesPerWave];
            {
                const float2 cn = w.c_norm[pc.base / kTileRows + min(k0 + lane, c1 - 1)];
#pragma unroll
                for (int t = 0; t < kTilesPerWave; ++t) {
                    const float tl = __shfl(lo, t * kTileCols, kWave), th = __shfl(hi, t * kTileCols, kWave);
                    need[t] = ballot(k0 + lane < c1 && cn.x <= th && cn.y >= tl);
                }
            }
            const uint64_t all = (need[0] & need[1]) & (need[2] & need[3]);
#pragma unroll
            for (int t = 0; t < kTilesPerWave; ++t)
                if (kCount) done += __popcll(need[t]);
            for_chunks(b, k0, (need[0] | need[1]) | (need[2] | need[3]), lane, [&](const ChunkRegs& a, int k) {
                i32x4 s[kTilesPerWave];
                uint64_t has[kTilesPerWave];
                if ((all >> (k - k0)) & 1) {
                    group_scores(a, q, s);
#pragma unroll
                    for (int t = 0; t < kTilesPerWave; ++t)
                        has[t] = ballot(max(max(s[t][0], s[t][1]), max(s[t][2], s[t][3])) >= least[t]);
                } else {
#pragma unroll
                    for (int t = 0; t < kTilesPerWave; ++t) {
                        has[t] = 0ull;
                        if (!((need[t] >> (k - k0)) & 1)) continue;  // uniform
                        s[t] = tile_scores(a, q.h[t], q.l[t]);
                        has[t] = ballot(max(max(s[t][0], s[t][1]), max(s[t][2], s[t][3])) >= least[t]);
                    }
                }
                if ((has[0] | has[1]) | (has[2] | has[3])) {
                    const uint32_t where =
                        static_cast<uint32_t>(k * kTileRows + 4 * (lane >> 4)) | (static_cast<uint32_t>(lane & 15) << 26);
#pragma unroll
                    for (int t = 0; t < kTilesPerWave; ++t) {
                        if (!has[t]) continue;  // uniform
                        if ((has[t] >> lane) & 1) {
                            const int at = n_hit + lanes_below(has[t]);
                            s_hit[wv][at] = s[t];
                            s_at[wv][at] = where + (static_cast<uint32_t>(t * kTileCols) << 26);
                        }
                        n_hit += __popcll(has[t]);
                    }
                    if (n_hit > kStage - kTilesPerWave * kWave) hand_out();
                }
            });
        }
        if (n_hit) hand_out();
    }
    if (kCount) count_work(work, done);
}

// ------------------------------------------------------ exact re-scoring --

// The plain FP64 sum in dimension order; the loads of eight dimensions issue
// together (the sum keeps its order).
__device__ __forceinline__ double exact_d2(const float* __restrict__ x, const float* __restrict__ y, int dim) {
#pragma clang fp contract(off)
    double acc = 0.0;
    int t = 0;
    for (; t + 8 <= dim; t += 8) {
        float xs[8], ys[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            xs[u] = x[t + u];
            ys[u] = y[t + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double df = static_cast<double>(xs[u]) - static_cast<double>(ys[u]);
            acc = acc + df * df;
        }
    }
    for (; t < dim; ++t) {
        const double df = static_cast<double>(x[t]) - static_cast<double>(y[t]);
        acc = acc + df * df;
    }
    return acc;
}

// Combines two (best, its index, second) triples: smallest (b1, j1) first;
// the second is the smallest of the other best and both seconds.
__device__ __forceinline__ void combine_best(double& b1, int& j1, double& b2, double ob1, int oj1, double ob2) {
    const bool mine = (b1 < ob1) || (b1 == ob1 && j1 < oj1);
    const double nb2 = mine ? fmin(b2, ob1) : fmin(ob2, b1);
    if (!mine) {
        b1 = ob1;
        j1 = oj1;
    }
    b2 = nb2;
}

constexpr int kScoreLanes = 16;  // lanes per query
constexpr int kRegList = 4;      // list entries per lane kept in registers
constexpr int kLongList = kScoreLanes * kRegList;  // longer lists go to whole wavefronts

// The exact nearest and second nearest row of one query from its list of m
// rows (plus the partner's rows out of range), by W lanes (gl: lane in the
// group), every lane with the result; `scored` is the number of exact scores.
struct Nearest {
    double b1, b2;
    int j1, scored;
};
template <int W>
__device__ __forceinline__ Nearest score_query(const MatchSet& qs, const MatchSet& ps, const SetPlan& qc,
                                               const SetPlan& pc, int dim, double scale, const MatchWs& w, int64_t slot,
                                               int m, int cap, int gl, int* rows) {
    const uint2* src = w.pool + slot * cap;
    const int own = w.half[slot] + 1;
    const double e = static_cast<double>(w.err[slot]);
    uint2 ent[kRegList];
    int m1 = kNoRow, m2 = kNoRow;
#pragma unroll
    for (int u = 0; u < kRegList; ++u) {
        const int k = u * W + gl;
        ent[u] = k < m ? src[k] : make_uint2(0u, static_cast<uint32_t>(kNoRow));
    }
    const auto see = [&](int v) {
        m2 = max(min(m1, v), m2);
        m1 = max(m1, v);
    };
#pragma unroll
    for (int u = 0; u < kRegList; ++u) see(static_cast<int>(ent[u].y));
    for (int k = kRegList * W + gl; k < m; k += W) see(static_cast<int>(src[k].y));
#pragma unroll
    for (int d = 1; d < W; d <<= 1) {
        const int o1 = __shfl_xor(m1, d, W), o2 = __shfl_xor(m2, d, W);
        m2 = max(min(m1, o1), max(m2, o2));
        m1 = max(m1, o1);
    }
    const int least =
        max(least_score(m2 == kNoRow ? m2 : m2 + own, e + most_err(dim)) - own, INT_MIN + 1);
    const float* y = set_row(qs, w.perm[slot], dim);
    const int32_t* perm = w.perm + pc.base;  // listed rows are places in the norm order
    Nearest o{INFINITY, INFINITY, INT_MAX, 0};
    const auto take = [&](int j) {
        const double d = exact_d2(set_row(ps, j, dim), y, dim);
        if (d < o.b1 || (d == o.b1 && j < o.j1 && d < INFINITY)) {  // an infinite distance is none
            o.b2 = o.b1;
            o.b1 = d;
            o.j1 = j;
        } else if (d < o.b2) {
            o.b2 = d;
        }
    };
    // What the bound leaves is gathered first, so that the lanes score it side by side: a
    // lane's own four entries would run one after another (16 LiDAR pairs 253 -> 221 us, 64
    // pairs 655 -> 600, 13,000 x 15,400 rows 23.6 -> 18.3; a single LiDAR pair the same).
    const int lane0 = static_cast<int>(threadIdx.x) % kWave - gl;
    const uint64_t below = (uint64_t{1} << gl) - 1;
    const auto score_left = [&]() {
        int n = 0;
#pragma unroll
        for (int u = 0; u < kRegList; ++u) {
            const bool left = static_cast<int>(ent[u].y) >= least;
            const uint64_t who = __ballot(left) >> lane0 & (~uint64_t{0} >> (kWave - W));
            if (left) rows[n + __popcll(who & below)] = perm[ent[u].x];
            n += __popcll(who);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int k = gl; k < n; k += W) {
            ++o.scored;
            take(rows[k]);
        }
        __builtin_amdgcn_wave_barrier();
    };
    score_left();
    for (int k0 = kRegList * W; k0 < m; k0 += kRegList * W) {
#pragma unroll
        for (int u = 0; u < kRegList; ++u) {
            const int k = k0 + u * W + gl;
            ent[u] = k < m ? src[k] : make_uint2(0u, static_cast<uint32_t>(kNoRow));
        }
        score_left();
    }
    const auto merge = [&]() {
#pragma unroll
        for (int d = 1; d < W; d <<= 1) {
            const double o1 = __shfl_xor(o.b1, d, W), o2 = __shfl_xor(o.b2, d, W);
            const int oj = __shfl_xor(o.j1, d, W);
            combine_best(o.b1, o.j1, o.b2, o1, oj, o2);
        }
    };
    merge();
    // the partner's rows out of range: as integers farther from the centre than kRange, and
    // rounding may have lengthened them by as much as it moves any row, so farther from the
    // query than kRange less that much, less the query's own distance from the centre
    if (pc.n_out > 0) {
        const double far = kRange - most_err(dim) - (sqrt(-2.0 * static_cast<double>(own) + 2.0) + e);
        const double gap = far * (1.0 - 1e-6) * scale;
        if (!(gap > 0.0 && o.b2 < gap * gap)) {
            if (gl != 0) {  // the merged triple stays on the first lane only
                o.b1 = o.b2 = INFINITY;
                o.j1 = INT_MAX;
            }
            for (int k = gl; k < pc.n_out; k += W) take(w.out_list[pc.base + k]);
            merge();
        }
    }
#pragma unroll
    for (int d = 1; d < W; d <<= 1) o.scored += __shfl_xor(o.scored, d, W);
    return o;
}

// 16 lanes per query, a block per quarter of a group: the two best scores of
// the query's list bound it again, and what is left is scored exactly, a row
// per lane.  Queries with longer lists are listed for whole wavefronts, those
// out of range or with an overflowed list for the exact scan (both in
// score_rest).  Latency bound (a chain of list, row and descriptor loads per
// query), so every query is in flight at once, and seven wavefronts per SIMD (72
// registers instead of 86): a LiDAR pair 28 -> 25 us, 64 pairs 696 -> 663, 100,000
// rows 157 -> 143; with 64 registers a pair took 34.
__global__ __launch_bounds__(kBlock, 7) void score_lists(const MatchSet* __restrict__ sets, SetPlan* plan, int n_sets,
                                                      int dim, const int32_t* __restrict__ list,
                                                      const PairScale* __restrict__ pp, MatchWs w, MatchCtl* ctl,
                                                      const DevStatus* __restrict__ st) {
    constexpr int kPerBlock = kBlock / kScoreLanes;
    constexpr int kParts = kGroup / kPerBlock;
    __shared__ int s_more;
    __shared__ int s_rows[kPerBlock][kScoreLanes * kRegList];
    if (st->err_capacity) return;
    const int total = ctl->groups * kParts;
    const int cap = ctl->cap;
    const int gl = threadIdx.x % kScoreLanes;
    for (int it = blockIdx.x; it < total; it += gridDim.x) {
        const int gr = it / kParts;
        const int c = find_set(n_sets, gr, [&](int s) { return static_cast<int64_t>(plan[s].grp_off); });
        const SetPlan qc = plan[c], pc = plan[c ^ 1];
        if (threadIdx.x == 0) s_more = 0;
        __syncthreads();
        const int i = (gr - qc.grp_off) * kGroup + (it % kParts) * kPerBlock +
                      static_cast<int>(threadIdx.x) / kScoreLanes;
        if (i < qc.nq) {  // uniform over the query's lanes
            const int slot = list ? list[qc.base + i] : qc.base + i;
            const int found = w.cnt[slot];
            if (w.err[slot] < 0.0f || found > cap) {
                if (gl == 0) {
                    // listed in the set's own range (in any order: each query's scan stands alone)
                    w.fb_list[qc.base + atomicAdd(&plan[c].n_open, 1)] = slot;
                    w.long_list[w.slot_cap - 1 - atomicAdd(&ctl->open, 1)] = slot;  // and from the end of the other
                    w.cnt[slot] = 0;  // counts the finished segments from here on
                    atomicAdd(&s_more, 1);
                }
            } else if (found > kLongList) {
                if (gl == 0) w.long_list[atomicAdd(&ctl->n_long, 1)] = slot;
            } else {
                const Nearest o = score_query<kScoreLanes>(sets[c], sets[c ^ 1], qc, pc, dim, pp[c >> 1].scale, w, slot,
                                                           found, cap, gl,
                                                           s_rows[threadIdx.x / kScoreLanes]);
                if (gl == 0) {
                    const int64_t at = qc.base + w.perm[slot];
                    w.nn[at] = o.j1 == INT_MAX ? -1 : o.j1;
                    w.best[at] = o.b1;
                    w.second[at] = o.b2;
                    if (o.scored > 4) atomicAdd(&s_more, 1);
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0 && s_more) atomicAdd(&w.fb_part[c * kFbParts + it % kFbParts], s_more);
        __syncthreads();
    }
}

constexpr int kFewOpen = 16;  // up to here the exact scans run a wavefront per query and segment
constexpr int kXSegMax = 256;  // row segments per group of the exact scan
// Rows of a segment from which a bound on the norms is looked for: it costs 3 us, as much
// as a tile of 128 rows (two pairs of 1,849 raw points a cloud: 41 us, with it 44).
constexpr int kBoundRows = 512;

// Row segments of the exact scan of F listed queries in `groups` groups:
// enough items for the chip, as many as the partial buffer holds.
__device__ __forceinline__ int exact_segs(int64_t F, int64_t groups, int64_t part_cap) {
    const int64_t want = max(static_cast<int64_t>(8), kRestBlocks / max(groups, static_cast<int64_t>(1)));
    const int64_t s = min(min(want, part_cap / (3 * F)), static_cast<int64_t>(kXSegMax));
    return static_cast<int>(s < 1 ? 1 : s);
}

// What score_lists left.  First the queries with long lists, a wavefront each.
// Then the queries listed for the exact scan.  Up to kFewOpen of them (rows out
// of range, as a rule) take a wavefront per query and segment, reading the rows
// from cache; the form for more shares each row among 64 queries:
// exact FP64 scans for the listed queries: plan[c].n_open entries of set c from
// fb_list[plan[c].base] on, in groups that never span two sets.  A work item is
// (group of up to 64 entries, row segment): the lanes of every wave hold the
// entries in registers as FP64, padded with zeros to 4 KS values, the partner rows
// of the segment stream through LDS as FP64 with the same zero padding (a padded
// term adds an exact zero), and each wave scores its share of the rows, ascending,
// two at a time, with the plain FP64 sum in dimension order.  FP64 issue bounds it,
// so a group of up to 8, 16 or 32 entries gives each one 8, 4 or 2 lanes, with
// rows of their own: a batch's sets have about seven such entries each, and a lane
// an entry left nine tenths of the wavefront idle (64 pairs 1,020 -> 761 us, 16
// pairs 244 -> 213, 100,000 rows 273 -> 244).
// A group whose entries are all there for an overflowed list takes the rows in norm
// order and passes over the tiles that none of them can reach by their norms, as the
// sweep does (a cluster of three tenths of 13,015 x 15,401 rows, closer together than
// the integers resolve: 1,170 -> 800 us for the call); the groups of a segment go to
// neighbouring blocks, so that a block's next item is of another segment (where the
// cluster lies in the order made some of them long: scan of six tenths 1,320 -> 1,180
// us).  Another group reads every row, as they lie.
// The lanes and waves of an entry merge their (best, index, second) and write them as
// the segment's partial result.  The block that finishes a group's last segment
// (counted in grp_done, which comes in cleared) merges the group's partials in segment
// order into nn, best and second, and resets the count.
template <int KS>
__global__ __launch_bounds__(kBlock) void score_rest(const MatchSet* __restrict__ sets, SetPlan* plan, int n_sets,
                                                     int dim, const PairScale* __restrict__ pp, MatchWs w,
                                                     const MatchCtl* __restrict__ ctl) {
#pragma clang fp contract(off)
    constexpr int kD = 4 * KS;                   // padded row length
    constexpr int kXRows = KS <= 9 ? 128 : 64;   // partner rows per LDS tile
    __shared__ __attribute__((aligned(16))) double s_x[kXRows * kD];
    __shared__ const float* s_row[kXRows];
    __shared__ int s_id[kXRows];
    __shared__ double s_b1[kBlock], s_b2[kBlock];
    __shared__ int s_j1[kBlock];
    __shared__ int s_last;
    __shared__ int s_pre[kPlanThreads + 1];   // the sets' first entries
    __shared__ int s_gpre[kPlanThreads + 1];  // and first groups
    constexpr int kWaves = kBlock / kWave;
    const int L = threadIdx.x % kWave;
    const int wv = threadIdx.x / kWave;
    const int64_t F = ctl->open;
    for (int k = global_wave(); k < ctl->n_long; k += wave_count()) {  // the long lists, a wavefront each
        const int64_t slot = w.long_list[k];
        const int c = find_set(n_sets, slot, [&](int s) { return static_cast<int64_t>(plan[s].base); });
        const Nearest o = score_query<kWave>(sets[c], sets[c ^ 1], plan[c], plan[c ^ 1], dim, pp[c >> 1].scale, w, slot,
                                             w.cnt[slot], ctl->cap, L,
                                             reinterpret_cast<int*>(s_x) + wv * kWave * kRegList);
        if (L == 0) {
            const int64_t at = plan[c].base + w.perm[slot];
            w.nn[at] = o.j1 == INT_MAX ? -1 : o.j1;
            w.best[at] = o.b1;
            w.second[at] = o.b2;
            if (o.scored > 4) atomicAdd(&w.fb_part[c * kFbParts + k % kFbParts], 1);
        }
    }
    if (F <= kFewOpen) {
        // few: a wavefront per query and segment of the partner's rows, a row per lane at a
        // time; the one that finishes a query's last segment merges the partials
        const int S = F > 0 ? static_cast<int>(min(static_cast<int64_t>(kRestBlocks * kWaves) / F, static_cast<int64_t>(kWave))) : 1;
        double* const pb1 = w.part;
        double* const pb2 = w.part + F * S;
        int32_t* const pj1 = reinterpret_cast<int32_t*>(w.part + 2 * F * S);
#pragma unroll 1
        for (int64_t it = global_wave(); it < F * S; it += wave_count()) {
            const int64_t f = it / S;
            const int sg = static_cast<int>(it - f * S);
            const int64_t slot = w.long_list[w.slot_cap - 1 - f];
            const int c = find_set(n_sets, slot, [&](int s) { return static_cast<int64_t>(plan[s].base); });
            const MatchSet ps = sets[c ^ 1];
            const int row = w.perm[slot];
            const float* y = set_row(sets[c], row, dim);
            const int np = plan[c ^ 1].n, len = (np + S - 1) / S;
            const int end = min(np, (sg + 1) * len);
            double b1 = INFINITY, b2 = INFINITY;
            int j1 = INT_MAX;
#pragma unroll 1
            for (int j = sg * len + L; j < end; j += kWave) {
                const double d = exact_d2(set_row(ps, j, dim), y, dim);
                if (d < b1) {
                    b2 = b1;
                    b1 = d;
                    j1 = j;
                } else if (d < b2) {
                    b2 = d;
                }
            }
            const auto merge = [&]() {
#pragma unroll 1
                for (int d = 1; d < kWave; d <<= 1) {
                    const double o1 = __shfl_xor(b1, d, kWave), o2 = __shfl_xor(b2, d, kWave);
                    const int oj = __shfl_xor(j1, d, kWave);
                    combine_best(b1, j1, b2, o1, oj, o2);
                }
            };
            merge();
            int last = 0;
            if (L == 0) {
                pb1[it] = b1;
                pb2[it] = b2;
                pj1[it] = j1;
                __threadfence();
                last = atomicAdd(&w.cnt[slot], 1) == S - 1;
            }
            if (!__shfl(last, 0, kWave)) continue;
            __threadfence();  // the other segments' partials are visible from here on
            b1 = b2 = INFINITY;
            j1 = INT_MAX;
            if (L < S) {
                b1 = pb1[f * S + L];
                b2 = pb2[f * S + L];
                j1 = pj1[f * S + L];
            }
            merge();
            if (L == 0) {
                const int64_t at = plan[c].base + row;
                w.nn[at] = j1 == INT_MAX ? -1 : j1;
                w.best[at] = b1;
                w.second[at] = b2;
            }
        }
        return;
    }
    __syncthreads();  // s_x held the long lists' rows
    for (int i = threadIdx.x; i < kXRows * (kD - dim); i += kBlock)  // the padding, zero for good
        s_x[(i / (kD - dim)) * kD + dim + i % (kD - dim)] = 0.0;
    if (wv == 0) {  // lane L sums sets [kPer L, kPer (L + 1)), then the wave scans the sums
        constexpr int kPer = (kPlanThreads + kWave) / kWave;
        int v[kPer];
        int sum = 0, gsum = 0;
        for (int k = 0; k < kPer; ++k) {
            const int c = L * kPer + k;
            v[k] = c < n_sets ? plan[c].n_open : 0;
            sum += v[k];
            gsum += (v[k] + kWave - 1) / kWave;
        }
        int run = wave_incl_scan(sum) - sum;
        int grun = wave_incl_scan(gsum) - gsum;
        for (int k = 0; k < kPer; ++k) {
            const int c = L * kPer + k;
            if (c <= n_sets) {
                s_pre[c] = run;
                s_gpre[c] = grun;
            }
            run += v[k];
            grun += (v[k] + kWave - 1) / kWave;
        }
    }
    __syncthreads();
    const int64_t groups = s_gpre[n_sets];
    const int S = exact_segs(F, groups, w.part_cap);
    double* const part = w.part;
    double* pb1 = part;
    double* pb2 = part + F * S;
    int32_t* pj1 = reinterpret_cast<int32_t*>(part + 2 * F * S);
    const int64_t items = groups * S;
    for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
        const int sg = static_cast<int>(item / groups);
        const int64_t g = item - sg * groups;
        int lo = 0, hi = n_sets - 1;  // the group's set: the last whose first group is <= g
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_gpre[mid] <= g) lo = mid;
            else hi = mid - 1;
        }
        const int c = lo, p = lo ^ 1;
        // a lane's entry of the group (dense index e into the partials), its slot and its row of R
        const int first = static_cast<int>(g - s_gpre[c]) * kWave;
        const int n_here = s_pre[c + 1] - s_pre[c] - first;  // at least 1
        const int Q = n_here > 32 ? 64 : n_here > 16 ? 32 : n_here > 8 ? 16 : 8;
        const int R = kWave / Q, sub = L / Q;
        const int local = first + (L & (Q - 1));
        const bool have = local < s_pre[c + 1] - s_pre[c];
        const int64_t e = s_pre[c] + local;
        const int64_t slot = have ? w.fb_list[plan[c].base + local] : plan[c].base;
        const float err = w.err[slot], nu = w.nu[slot];
        double y[kD];
        {
            const float* yr = set_row(sets[c], w.perm[slot], dim);
#pragma unroll
            for (int t = 0; t < kD; ++t) {
                const double v = yr[min(t, dim - 1)];  // never predicated: all loads in flight
                y[t] = t < dim ? v : 0.0;
            }
        }
        // the norms that the entries of a group may need, when all are there for their lists: what
        // the first of the rows on them say
        float from = -INFINITY, upto = INFINITY;
        const int np = plan[p].n;
        int len = (np + S - 1) / S;
        if (len >= kBoundRows && !ballot(have && err < 0.0f)) {  // uniform in the block, and over the group's segments
            int v[kMinCap], m1 = kNoRow, m2 = kNoRow;
#pragma unroll
            for (int k = 0; k < kMinCap; ++k) v[k] = static_cast<int>(w.pool[slot * ctl->cap + k].y);
#pragma unroll
            for (int k = 0; k < kMinCap; ++k) {
                m2 = med3(m1, m2, v[k]);
                m1 = max(m1, v[k]);
            }
            const float reach = reach_of(m2 == kNoRow ? m2 : m2 + w.half[slot] + 1,
                                         static_cast<double>(err) + most_err(dim), pp[c >> 1].scale);
            from = have ? nu * (1.0f - kNormSlack) - reach : INFINITY;
            upto = have ? nu * (1.0f + kNormSlack) + reach : -INFINITY;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                from = fminf(from, __shfl_xor(from, d, kWave));
                upto = fmaxf(upto, __shfl_xor(upto, d, kWave));
            }
        }
        double b1 = INFINITY, b2 = INFINITY;
        int j1 = INT_MAX;
        {
            const int base = plan[p].base;
            const bool bounded = from > -INFINITY;
            if (bounded) len = (len + kTileRows - 1) / kTileRows * kTileRows;  // whole chunks
            const int r_begin = min(np, sg * len), r_end = min(np, r_begin + len);
            // rows in norm order where some can be passed over, else as they lie
            const auto row_at = [&](int r) {
                const int at = min(r + static_cast<int>(threadIdx.x) % kXRows, np - 1);
                return bounded ? w.perm[base + at] : at;
            };
            const auto norms_at = [&](int r) {
                const int at = min(r + L % (kXRows / kTileRows) * kTileRows, np - 1);
                return bounded ? w.c_norm[(base + at) / kTileRows] : make_float2(0.f, 0.f);
            };
            int next = row_at(r_begin);
            float2 next_norms = norms_at(r_begin);
            for (int r0 = r_begin; r0 < r_end; r0 += kXRows) {
                const int nr = min(kXRows, r_end - r0), j = next;
                const float2 cn = next_norms;
                next = row_at(r0 + kXRows);  // a tile ahead: the rows' addresses hang on it
                next_norms = norms_at(r0 + kXRows);
                if (bounded && !ballot(cn.x <= upto && cn.y >= from)) continue;  // none of the rows is needed
                __syncthreads();
                // the tile's rows: their addresses first, then all values by all threads,
                // eight loads in flight per thread
                if (static_cast<int>(threadIdx.x) < nr) {
                    s_id[threadIdx.x] = j;
                    s_row[threadIdx.x] = set_row(sets[p], j, dim);
                }
                __syncthreads();
                const int n_el = nr * dim;
                for (int e0 = static_cast<int>(threadIdx.x); e0 < n_el; e0 += 8 * kBlock) {
                    float v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int e = e0 + u * kBlock;
                        v[u] = e < n_el ? s_row[e / dim][e % dim] : 0.0f;
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int e = e0 + u * kBlock;
                        if (e < n_el) s_x[(e / dim) * kD + e % dim] = static_cast<double>(v[u]);
                    }
                }
                __syncthreads();
                {
                    const auto take = [&](double acc, int at) {
                        if (!(acc <= b2)) return;
                        const int j = s_id[at];
                        if (acc < b1 || (acc == b1 && j < j1 && acc < INFINITY)) {  // an infinite distance is none
                            b2 = b1;
                            b1 = acc;
                            j1 = j;
                        } else if (acc < b2) {
                            b2 = acc;
                        }
                    };
                    for (int rw = wv * R; rw < nr; rw += 2 * kWaves * R) {  // wave-uniform
                        const int ra = rw + sub, rb = ra + kWaves * R;
                        const double2* xa = reinterpret_cast<const double2*>(s_x + min(ra, nr - 1) * kD);
                        const double2* xb = reinterpret_cast<const double2*>(s_x + min(rb, nr - 1) * kD);
                        double a = 0.0, b = 0.0;
#pragma unroll
                        for (int t = 0; t < kD / 2; ++t) {
                            const double2 va = xa[t], vb = xb[t];
                            const double da0 = va.x - y[2 * t], db0 = vb.x - y[2 * t];
                            a = a + da0 * da0;
                            b = b + db0 * db0;
                            const double da1 = va.y - y[2 * t + 1], db1 = vb.y - y[2 * t + 1];
                            a = a + da1 * da1;
                            b = b + db1 * db1;
                        }
                        if (ra < nr) take(a, ra);
                        if (rb < nr) take(b, rb);
                    }
                }
            }
        }
        // the lanes of one entry, then the waves
        const auto merge_rows = [&]() {
#pragma unroll 1
            for (int d = Q; d < kWave; d <<= 1) {
                const double o1 = __shfl_xor(b1, d, kWave), o2 = __shfl_xor(b2, d, kWave);
                const int oj = __shfl_xor(j1, d, kWave);
                combine_best(b1, j1, b2, o1, oj, o2);
            }
        };
        merge_rows();
        s_b1[threadIdx.x] = b1;
        s_b2[threadIdx.x] = b2;
        s_j1[threadIdx.x] = j1;
        __syncthreads();
        if (wv == 0 && have && sub == 0) {
            for (int o = 1; o < kWaves; ++o)
                combine_best(b1, j1, b2, s_b1[o * kWave + L], s_j1[o * kWave + L], s_b2[o * kWave + L]);
            pb1[sg * F + e] = b1;
            pb2[sg * F + e] = b2;
            pj1[sg * F + e] = j1;
        }
        // wave 0 wrote the partials: it publishes them and counts the segment
        if (wv == 0) {
            __threadfence();
            if (L == 0) s_last = atomicAdd(&w.grp_done[g], 1) == S - 1;
        }
        __syncthreads();
        if (s_last) {  // uniform: the group's last segment; the partials dealt to the entry's lanes of all waves
            __threadfence();  // the other segments' partials are visible from here on
            b1 = b2 = INFINITY;
            j1 = INT_MAX;
            if (have) {
                // sixteen segments' loads in flight: the partials come from beyond the L2
                for (int k0 = wv * R + sub; k0 < S; k0 += 16 * kWaves * R) {
                    double o1[16], o2[16];
                    int oj[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) {
                        const int64_t at = static_cast<int64_t>(min(k0 + u * kWaves * R, S - 1)) * F + e;
                        o1[u] = pb1[at];
                        o2[u] = pb2[at];
                        oj[u] = pj1[at];
                    }
#pragma unroll
                    for (int u = 0; u < 16; ++u)
                        if (k0 + u * kWaves * R < S) combine_best(b1, j1, b2, o1[u], oj[u], o2[u]);
                }
            }
            merge_rows();
            s_b1[threadIdx.x] = b1;
            s_b2[threadIdx.x] = b2;
            s_j1[threadIdx.x] = j1;
            __syncthreads();
            if (wv == 0) {
                for (int o = 1; o < kWaves; ++o)
                    combine_best(b1, j1, b2, s_b1[o * kWave + L], s_j1[o * kWave + L], s_b2[o * kWave + L]);
                if (have && sub == 0) {
                    const int64_t at = plan[c].base + w.perm[slot];
                    w.nn[at] = (j1 == INT_MAX) ? -1 : j1;
                    w.best[at] = b1;
                    w.second[at] = b2;
                }
                if (L == 0) w.grp_done[g] = 0;  // ready for a later scan on this workspace
            }
        }
        __syncthreads();
    }
}

// --------------------------------------------------- matching back, output --

// One-sided form: the rows that are some query's nearest neighbour, each listed
// once (its nearest neighbour goes from -1, none, to -2, claimed; the matching
// back answers every listed row), in no particular order, in its set's own
// range of img_list, counted in plan[c].n_img.
__global__ __launch_bounds__(kBlock) void image_lists(SetPlan* plan, int n_sets, MatchWs w,
                                                      const MatchCtl* __restrict__ ctl,
                                                      const DevStatus* __restrict__ st) {
    if (st->err_capacity) return;
    const int64_t total = ctl->slots;
    const int64_t gs = static_cast<int64_t>(gridDim.x) * kBlock;
    const int lane = lane_id();
    // wave-uniform trip count: the appends are counted once per wave and set
    for (int64_t w0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x - lane; w0 < total; w0 += gs) {
        const int64_t slot = w0 + lane;
        bool claim = false;
        int p = 0, j = 0;
        if (slot < total) {
            const int c = find_set(n_sets, slot, [&](int s) { return static_cast<int64_t>(plan[s].base); });
            const int i = static_cast<int>(slot) - plan[c].base;
            if (i < plan[c].nq && (c ^ 1) < n_sets) {
                j = w.nn[plan[c].base + w.perm[slot]];  // in norm order, so that the images come in it too
                p = c ^ 1;
                if (j >= 0) claim = atomicCAS(&w.nn[plan[p].base + j], -1, -2) == -1;
            }
        }
        uint64_t pending = ballot(claim);
        int k = 0;
        while (pending) {
            const int lead = __ffsll(static_cast<unsigned long long>(pending)) - 1;
            const int pl = __shfl(p, lead, kWave);
            const uint64_t same = ballot(claim && p == pl);
            int at = 0;
            if (lane == lead) at = atomicAdd(&plan[pl].n_img, __popcll(same));
            at = __shfl(at, lead, kWave);
            if (claim && p == pl) k = at + lanes_below(same);
            pending &= ~same;
        }
        if (claim) w.img_list[plan[p].base + k] = plan[p].base + w.inv[plan[p].base + j];
    }
}

// The mutual test, the correspondences in order of the source row and the
// pair's counts, in one launch: a block takes a tile of kEmitTile source rows
// (tickets in launch order), and the tiles of a pair are chained through
// look-back words (zeroed by match_round), so that a chain is one set long.
__global__ __launch_bounds__(kBlock) void match_emit(const MatchSet* __restrict__ sets,
                                                     const SetPlan* __restrict__ plan, int n_pairs, MatchWs w,
                                                     const MatchCtl* __restrict__ ctl,
                                                     const PairOutDev* __restrict__ outs, DevStatus* st,
                                                     int64_t* __restrict__ counts, int stride,
                                                     const CloudState* __restrict__ cs, int64_t nnz_cap) {
    constexpr int kItems = kEmitTile / kBlock;
    __shared__ int s_tile, s_wave[kBlock / kWave];
    __shared__ int64_t s_prefix;
    const int total = ctl->emit_tiles;
    const bool empty = st->err_capacity != 0;  // nothing was matched
    while (true) {
        if (threadIdx.x == 0) s_tile = look_back_ticket(w.emit_status, total);
        __syncthreads();
        const int tile = s_tile;
        if (tile >= total) break;  // uniform
        const int pr = find_set(n_pairs, tile, [&](int s) { return static_cast<int64_t>(plan[2 * s].emit_off); });
        const int off = plan[2 * pr].emit_off;
        const int a0 = plan[2 * pr].base, b0 = plan[2 * pr + 1].base;
        const int na = plan[2 * pr].n, lt = tile - off;
        const int first = lt * kEmitTile + static_cast<int>(threadIdx.x) * kItems;
        int to[kItems], cnt = 0;
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
            to[u] = (!empty && first + u < na) ? w.nn[a0 + first + u] : -1;
        }
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
            if (to[u] >= 0 && w.nn[b0 + to[u]] != first + u) to[u] = -1;
            cnt += to[u] >= 0 ? 1 : 0;
        }
        const int wv = threadIdx.x / kWave;
        const int incl = wave_incl_scan(cnt);
        if (lane_id() == kWave - 1) s_wave[wv] = incl;
        __syncthreads();
        int before = 0, sum = 0;
#pragma unroll
        for (int k = 0; k < kBlock / kWave; ++k) {
            before += k < wv ? s_wave[k] : 0;
            sum += s_wave[k];
        }
        if (wv == 0) {
            const int64_t prefix = look_back(w.emit_status + off, lt, sum, &st->err_sync);
            if (threadIdx.x == 0) s_prefix = prefix;
        }
        __syncthreads();
        const PairOutDev o = outs[pr];
        const MatchSet a = sets[2 * pr], b = sets[2 * pr + 1];
        int64_t at = s_prefix + before + incl - cnt;
#pragma unroll
        for (int u = 0; u < kItems; ++u) {
            if (to[u] < 0) continue;
            if (at < o.cap) {
                const int j = first + u, i = to[u];
                o.pairs[2 * at] = (a.rows ? a.rows[j] : j) - a.row_base;
                o.pairs[2 * at + 1] = (b.rows ? b.rows[i] : i) - b.row_base;
                o.d1[at] = static_cast<float>(sqrt(w.best[a0 + j]));
                o.d2[at] = static_cast<float>(sqrt(w.second[a0 + j]));
            }
            ++at;
        }
        if (threadIdx.x == 0 && (lt + 1) * kEmitTile >= na) {  // the pair's last tile
            int64_t* q = counts + static_cast<int64_t>(pr) * stride;
            q[0] = s_prefix + sum;
            int more = 0;
            for (int k = 0; k < 2 * kFbParts; ++k) more += w.fb_part[2 * pr * kFbParts + k];
            q[5] = more;
            if (cs) {  // the batch form: sizes of the pair and its status
                q[1] = cs[2 * pr].kept_cnt;
                q[2] = cs[2 * pr + 1].kept_cnt;
                q[3] = cs[2 * pr].j_cnt;
                q[4] = cs[2 * pr + 1].j_cnt;
                q[7] = st->nnz;
                int64_t status = KMG_OK;
                if (st->err_sync) status = KMG_ERR_DEVICE;  // a bounded wait gave up (never expected)
                else if (st->err_range || (st->dense & 2)) status = KMG_ERR_RANGE;
                else if (st->err_capacity || st->nnz > nnz_cap) status = KMG_ERR_WORKSPACE;
                else if (q[0] > o.cap) status = KMG_ERR_CAPACITY;
                q[6] = status;
            }
        }
        __syncthreads();  // the shared words are free for the next tile
    }
}

}  // namespace

MatchWs carve_match(Carver& c, int n_sets, int64_t q_cap, int dim) {
    (void)dim;
    MatchWs w;
    w.q_cap = std::max<int64_t>(q_cap, 1);
    w.n_sets = n_sets;
    // every set starts on a chunk
    w.slot_cap = w.q_cap + static_cast<int64_t>(n_sets) * kTileRows;
    const int64_t grp_cap = w.q_cap / kGroup + n_sets;
    w.ctl = c.take<MatchCtl>(1);
    w.plan = c.take<SetPlan>(static_cast<size_t>(std::max(n_sets, 1)));
    w.pp = c.take<PairScale>(static_cast<size_t>(n_sets / 2 + 1));
    w.rows = c.take<unsigned char>(static_cast<size_t>(w.slot_cap) * kRowBytes);
    w.half = c.take<int>(static_cast<size_t>(w.slot_cap));
    w.nu = c.take<float>(static_cast<size_t>(w.slot_cap));
    w.c_norm = c.take<float2>(static_cast<size_t>(w.slot_cap / kTileRows + 1));
    w.perm = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    w.inv = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    // at most kTileWaves segments of the sample, and one more for each group
    w.s_best = c.take<int2>(static_cast<size_t>(grp_cap + kTileWaves) * kGroup);
    w.err = c.take<float>(static_cast<size_t>(w.slot_cap));
    w.cnt = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    // listed rows: kMinCap per slot whatever the size, up to kMaxCap from 128 MB more
    w.pool_cap = kMinCap * w.slot_cap + std::min<int64_t>((kMaxCap - kMinCap) * w.slot_cap, int64_t(1) << 24);
    w.pool = c.take<uint2>(static_cast<size_t>(w.pool_cap));
    // the exact scans' partials: (best, second, row) per listed query and segment
    w.part_cap = std::max<int64_t>(3 * w.slot_cap, int64_t(1) << 20);
    w.part = c.take<double>(static_cast<size_t>(w.part_cap));
    w.out_list = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    w.fb_list = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    w.long_list = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    w.img_list = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    w.nn = c.take<int32_t>(static_cast<size_t>(w.slot_cap));
    w.best = c.take<double>(static_cast<size_t>(w.slot_cap));
    w.second = c.take<double>(static_cast<size_t>(w.slot_cap));
    w.fb_part = c.take<int32_t>(static_cast<size_t>(n_sets) * kFbParts);
    w.grp_done = c.take<int32_t>(static_cast<size_t>(w.slot_cap / kWave + n_sets + 2));
    w.emit_status = c.take<uint64_t>(static_cast<size_t>(w.q_cap / kEmitTile + n_sets + 2));
    w.work = c.take<int64_t>(2 * kMaxWorkCounters);
    return w;
}

namespace {

// One phase: the planned queries (all rows of their sets, or the listed ones)
// through the sample pass, the sweep, the exact scores and the exact scans.
kmg_status match_queries(const MatchSet* sets, int n_sets, int dim, const int32_t* list, DevStatus* st,
                         const MatchWs& w, hipStream_t s) {
    {
        StageScope sc(ST_MATCH_TOPK, s);
        int64_t* const work = w.work + (list ? kMaxWorkCounters : 0);
        const auto sample = timer_on() ? &sample_tiles<true> : &sample_tiles<false>;
        const auto sweep = timer_on() ? &sweep_tiles<true> : &sweep_tiles<false>;
        sample<<<kTileBlocks, kBlock, 0, s>>>(w.plan, n_sets, dim, list, w.pp, w, w.ctl, st, work);
        KMG_TRY(launch_status());
        sweep<<<kTileBlocks, kBlock, 0, s>>>(w.plan, n_sets, dim, list, w.pp, w, w.ctl, st, work);
        KMG_TRY(launch_status());
        timer_note_work(work, kMaxWorkCounters);
    }
    StageScope sc(ST_MATCH_RESCORE, s);
    score_lists<<<grid_cap((w.q_cap / kGroup + n_sets) * (kGroup * kScoreLanes / kBlock), 1), kBlock, 0, s>>>(sets, w.plan, n_sets, dim, list, w.pp, w,
                                                                          w.ctl, st);
    KMG_TRY(launch_status());
    if (dim <= 36) score_rest<9><<<kRestBlocks, kBlock, 0, s>>>(sets, w.plan, n_sets, dim, w.pp, w, w.ctl);
    else score_rest<17><<<kRestBlocks, kBlock, 0, s>>>(sets, w.plan, n_sets, dim, w.pp, w, w.ctl);
    return launch_status();
}

// Products of a pair above which the one-sided form pays for its six more
// launches (about 30 us): a direction of 4e8 products takes about 60 us, and
// the matching back serves a quarter to a half of the larger set.
constexpr int64_t kOneSidedProducts = int64_t(1) << 29;

kmg_status match_sets(MatchSet* sets, int n_sets, int dim, int64_t products, const SinglePair& single, DevStatus* st,
                      const MatchWs& w, const PairOutDev* outs, int64_t* counts, int counts_stride, hipStream_t s,
                      const CloudState* cs, int64_t nnz_cap) {
    if (dim < 1 || dim > kMaxMatchDim) return KMG_ERR_ARG;
    const bool one_sided = tuning().match_form == 0 && products > kOneSidedProducts;
    {
        StageScope sc(ST_MATCH_PACK, s);
        const int order = static_cast<int>(std::min<int64_t>(w.q_cap / kSortTile + n_sets, kSortBlocks));
        match_plan<<<1 + n_sets / 2 + order, kPlanThreads, 0, s>>>(sets, n_sets, dim, one_sided ? 1 : 0, w.pool_cap,
                                                                   w.plan, w.ctl, w.pp, single, w, st);
        KMG_TRY(launch_status());
        match_round<<<grid_cap(w.slot_cap * 8, kBlock), kBlock, 0, s>>>(sets, w.plan, n_sets, dim, w.pp, w, w.ctl);
        KMG_TRY(launch_status());
    }
    KMG_TRY(match_queries(sets, n_sets, dim, nullptr, st, w, s));
    if (one_sided) {
        StageScope sc(ST_MATCH_IMAGE, s);
        image_lists<<<grid_cap(w.slot_cap, kBlock), kBlock, 0, s>>>(w.plan, n_sets, w, w.ctl, st);
        KMG_TRY(launch_status());
        match_plan_back<<<1, kPlanThreads, 0, s>>>(n_sets, w.plan, w.ctl, st);
        KMG_TRY(launch_status());
        KMG_TRY(match_queries(sets, n_sets, dim, w.img_list, st, w, s));
    }
    StageScope sc(ST_MATCH_MUTUAL, s);
    match_emit<<<grid_cap(w.q_cap / kEmitTile + n_sets / 2 + 1, 1), kBlock, 0, s>>>(
        sets, w.plan, n_sets / 2, w, w.ctl, outs, st, counts, counts_stride, cs, nnz_cap);
    return launch_status();
}

}  // namespace

kmg_status match_batch(MatchSet* sets, int n_sets, int dim, DevStatus* st, const MatchWs& w, const PairOutDev* outs,
                       int64_t* counts, int counts_stride, hipStream_t s, const CloudState* cs, int64_t nnz_cap) {
    if (n_sets < 2 || n_sets > kMaxClouds) return KMG_ERR_ARG;
    // the sizes are on the device: about an eighth of the raw points become rows
    const int64_t rows = w.q_cap / (8 * static_cast<int64_t>(n_sets)) + 1;
    return match_sets(sets, n_sets, dim, n_sets / 2 * rows * rows, SinglePair{}, st, w, outs, counts, counts_stride,
                      s, cs, nnz_cap);
}

// ---------------------------------------------------- single pair entry --

size_t match_ws(int64_t np, int64_t nq, int dim) {
    Carver c(nullptr, 0);
    c.take<DevStatus>(1);
    c.take<MatchSet>(2);
    c.take<int32_t>(2);
    c.take<PairOutDev>(1);
    c.take<int64_t>(8);
    carve_match(c, 2, np + nq, dim);
    return c.off;
}

kmg_status match(const float* dp, const int32_t* rp, int64_t np, const float* dq, const int32_t* rq, int64_t nq,
                 int dim, int32_t* pairs, float* d1, float* d2, int64_t cap, int64_t* n_pairs_host,
                 int64_t* n_fallback_host, void* ws, size_t ws_bytes, hipStream_t s) {
    Carver c(ws, ws_bytes);
    DevStatus* st = c.take<DevStatus>(1);
    MatchSet* sets = c.take<MatchSet>(2);
    int32_t* cnt = c.take<int32_t>(2);
    PairOutDev* outs = c.take<PairOutDev>(1);
    int64_t* counts = c.take<int64_t>(8);
    MatchWs w = carve_match(c, 2, np + nq, dim);
    if (!c.fits()) return KMG_ERR_WORKSPACE;
    *n_pairs_host = 0;
    if (n_fallback_host) *n_fallback_host = 0;
    if (np == 0 || nq == 0) return KMG_OK;
    SinglePair p{};
    p.on = 1;
    p.a = MatchSet{dp, rp, nullptr, 0, 0};
    p.b = MatchSet{dq, rq, nullptr, 0, 0};
    p.na = static_cast<int32_t>(np);
    p.nb = static_cast<int32_t>(nq);
    p.counts = cnt;
    p.out = PairOutDev{pairs, d1, d2, cap};
    p.out_dev = outs;
    KMG_TRY(match_sets(sets, 2, dim, np * nq, p, st, w, outs, counts, 8, s, nullptr, 0));
    int64_t hc[8];
    DevStatus hs;
    Report r;
    KMG_TRY(r.post(counts, sizeof(hc), st, sizeof(hs), s));
    KMG_TRY(r.wait(hc, &hs));
    timer_collect();
    if (hs.err_capacity) return KMG_ERR_WORKSPACE;
    if (hs.err_sync) return KMG_ERR_DEVICE;
    *n_pairs_host = hc[0];
    if (n_fallback_host) *n_fallback_host = hc[5];
    if (hc[0] > cap) return KMG_ERR_CAPACITY;
    return KMG_OK;
}

// The lengths the band_tile field of the tuning accepts: every length 1 .. 64,
// then four per octave up to 4096.
bool band_tile_candidate(int T) {
    if (T >= 1 && T <= 64) return true;
    for (int o = 64; o < 4096; o *= 2)
        for (int k = 1; k <= 4; ++k)
            if (T == o + o / 4 * k) return true;
    return false;
}

}  // namespace kmg
