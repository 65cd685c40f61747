// Downstream of matching (Section III-D): the ratio filter that keeps the
// N_tau correspondences with the lowest descriptor distance ratio, the
// pairwise-invariant compatibility graph of Eq. (3), and its maximum k-core.
//
// Ratio filter.  The key of correspondence e is its ratio d1/d2 in FP64 from
// the float32 distances (0 when both are 0, +inf when only d2 is 0); keys are
// non-negative, so their bit patterns order like the values.  Correspondences
// are ranked by (key, position) by counting, which is exact and needs no sort;
// the first N_tau ranks are the graph's vertices, vertex v = rank v.
//
// Graph.  Vertices u != v are adjacent iff | ||b_u - b_v|| - ||a_u - a_v|| |
// <= 2 beta, with both norms evaluated in FP64 as sqrt((dx dx + dy dy) + dz dz)
// from the float32 kept coordinates (contraction off).  One wavefront per
// row tests 64 columns at a time: a count pass, a scan, then a fill pass that
// writes every row ascending.
//
// k-core.  Core numbers by level-synchronous peeling in one block: at level
// k, every vertex whose remaining degree is <= k is removed (core number k)
// and its alive neighbours lose one degree, round after round until none is
// left at that level; then the level jumps to the smallest remaining degree.  Core numbers are unique, so the parallel order of
// removals cannot change them.  The maximum k-core is the set of vertices
// whose core number is the largest.
#include <climits>
#include <math.h>

#include "kmg_device.h"

namespace kmg {

namespace {

constexpr int kBlock = 256;
constexpr int kPeelThreads = 1024;
constexpr int kMaxKcore = KMG_MAX_KCORE_VERTICES;  // LDS: 4 + 2 + 2 bytes per vertex

// Also clears what the call counts in: the ranks, the degrees, the look-back
// words of their scan and the index flag.
__global__ __launch_bounds__(kBlock) void ratio_keys(const float* __restrict__ d1, const float* __restrict__ d2,
                                                     int64_t k, uint64_t* __restrict__ keys,
                                                     int32_t* __restrict__ rank, FillJobs fills) {
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; e < k;
         e += static_cast<int64_t>(gridDim.x) * kBlock) {
        const double a = d1[e], b = d2[e];
        const double r = b > 0.0 ? a / b : (a > 0.0 ? INFINITY : 0.0);
        keys[e] = static_cast<uint64_t>(__double_as_longlong(r));
        rank[e] = 0;
    }
    run_fill_jobs(fills);
}

// rank[e] = number of correspondences f ordered before e by (key, position).
// Block (x, y) counts, for the keys of tile x, the keys of tiles y, y + gy, ...
// (staged in LDS) that come first, and adds its counts with one atomic per key.
// Equal keys count where they lie before: all of a tile before x, none of one
// after it, so that only tile x itself compares positions.  The LDS reads of
// eight keys are in flight at a time (one at a time: 19 us for 2,780
// correspondences, now 9).
constexpr int kRankTiles = 64;  // y tiles of the counting grid

__global__ __launch_bounds__(kBlock) void rank_count(const uint64_t* __restrict__ keys, int64_t k,
                                                     int32_t* __restrict__ rank) {
    __shared__ uint64_t s_key[kBlock];
    const int64_t e = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const bool live = e < k;
    const uint64_t me = live ? keys[e] : 0ull;
    int cnt = 0;
    for (int64_t f0 = static_cast<int64_t>(blockIdx.y) * kBlock; f0 < k;
         f0 += static_cast<int64_t>(gridDim.y) * kBlock) {
        __syncthreads();
        // keys are at most the bits of +inf or NaN (below ~0): the places past the end count nowhere
        s_key[threadIdx.x] = f0 + threadIdx.x < k ? keys[f0 + threadIdx.x] : ~0ull;
        __syncthreads();
        const int64_t x0 = static_cast<int64_t>(blockIdx.x) * kBlock;
        if (f0 == x0) {
#pragma unroll 8
            for (int t = 0; t < kBlock; ++t) {
                const uint64_t o = s_key[t];
                cnt += (o < me || (o == me && t < static_cast<int>(threadIdx.x))) ? 1 : 0;
            }
        } else if (f0 < x0) {  // a whole tile: its last key is inside
#pragma unroll 8
            for (int t = 0; t < kBlock; ++t) cnt += s_key[t] <= me ? 1 : 0;
        } else {
#pragma unroll 8
            for (int t = 0; t < kBlock; ++t) cnt += s_key[t] < me ? 1 : 0;
        }
    }
    if (live && cnt) atomicAdd(rank + e, cnt);
}

// The first n_tau ranks: sel[rank] = e and vertex rank's coordinates.
// Correspondence indices outside the clouds set err and read point 0 instead.
__global__ __launch_bounds__(kBlock) void gather_vertices(const float* __restrict__ src, int64_t src_stride,
                                                          const float* __restrict__ tgt, int64_t tgt_stride,
                                                          const int32_t* __restrict__ pairs,
                                                          const int32_t* __restrict__ rank, int64_t k, int32_t n_tau,
                                                          int32_t* __restrict__ sel, float4* __restrict__ va,
                                                          float4* __restrict__ vb, int32_t* __restrict__ err) {
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; e < k;
         e += static_cast<int64_t>(gridDim.x) * kBlock) {
        const int v = rank[e];
        if (v >= n_tau) continue;
        sel[v] = static_cast<int32_t>(e);
        int i = pairs[2 * e], j = pairs[2 * e + 1];
        if (i < 0 || i >= src_stride || j < 0 || j >= tgt_stride) {
            atomicOr(err, 1);
            i = 0;
            j = 0;
        }
        va[v] = make_float4(src[i], src[src_stride + i], src[2 * src_stride + i], 0.0f);
        vb[v] = make_float4(tgt[j], tgt[tgt_stride + j], tgt[2 * tgt_stride + j], 0.0f);
    }
}

__device__ __forceinline__ double norm_between(float4 p, float4 q) {
#pragma clang fp contract(off)
    const double dx = static_cast<double>(p.x) - static_cast<double>(q.x);
    const double dy = static_cast<double>(p.y) - static_cast<double>(q.y);
    const double dz = static_cast<double>(p.z) - static_cast<double>(q.z);
    return sqrt((dx * dx + dy * dy) + dz * dz);
}

// Eq. (3) for vertices u != v.
__device__ __forceinline__ bool compatible(float4 au, float4 bu, float4 av, float4 bv, double two_beta) {
#pragma clang fp contract(off)
    const double da = norm_between(au, av);
    const double db = norm_between(bu, bv);
    return fabs(db - da) <= two_beta;
}

// The same decision from FP32 where it is certain: dx, dy, dz are rounded
// differences of FP32 coordinates and the norm's relative error is below 4e-7,
// so with 1e-6 (da + db) and the squares that underflow allowed for, only a
// pair within that of the threshold (one in some ten thousand), and what is
// not finite, takes the FP64 form (`sure` false).
__device__ __forceinline__ bool compatible_fp32(float4 au, float4 bu, float4 av, float4 bv, float two_beta,
                                                bool& sure) {
    const float ax = au.x - av.x, ay = au.y - av.y, az = au.z - av.z;
    const float bx = bu.x - bv.x, by = bu.y - bv.y, bz = bu.z - bv.z;
    const float da = sqrtf(fmaf(az, az, fmaf(ay, ay, ax * ax)));
    const float db = sqrtf(fmaf(bz, bz, fmaf(by, by, bx * bx)));
    const float gap = fabsf(db - da) - two_beta;
    sure = fabsf(gap) > fmaf(1e-6f, da + db + fabsf(two_beta), 1e-18f) && da + db < INFINITY;
    return gap < 0.0f;
}

// One wavefront per row.  Two FP64 square roots per pair, and the loads of one
// piece of 64 columns at a time, took 29 us (count) and 33 us (fill) for 2,780
// vertices; the FP32 decision with four pieces in flight takes 17 and 23.
template <bool kFill>
__global__ __launch_bounds__(kBlock) void graph_rows(const float4* __restrict__ va, const float4* __restrict__ vb,
                                                     int32_t n, double beta, int32_t* __restrict__ deg,
                                                     const int32_t* __restrict__ off, int32_t* __restrict__ adj) {
    constexpr int kCols = 4;  // 64-column pieces whose loads are in flight together
    const int lane = lane_id();
    const double two_beta = 2.0 * beta;
    const float two_beta_f = static_cast<float>(two_beta);
    for (int64_t u = global_wave(); u < n; u += wave_count()) {
        const float4 au = va[u], bu = vb[u];
        int found = 0;
        int32_t* out = kFill ? adj + off[u] : nullptr;
        for (int base = 0; base < n; base += kCols * kWave) {
            float4 av[kCols], bv[kCols];
#pragma unroll
            for (int k = 0; k < kCols; ++k) {
                const int vc = min(base + k * kWave + lane, n - 1);  // unconditional loads; the mask applies afterwards
                av[k] = va[vc];
                bv[k] = vb[vc];
            }
#pragma unroll
            for (int k = 0; k < kCols; ++k) {
                const int v = base + k * kWave + lane;
                bool sure;
                bool near = compatible_fp32(au, bu, av[k], bv[k], two_beta_f, sure);
                if (ballot(!sure)) near = compatible(au, bu, av[k], bv[k], two_beta);  // uniform
                const bool e = v < n && v != u && near;
                const uint64_t b = ballot(e);
                if (kFill && e) out[found + lanes_below(b)] = v;
                found += __popcll(b);
            }
        }
        if (!kFill && lane == 0) deg[u] = found;
    }
}

// Core numbers as the fixed point of the h-index operator: start from h = degree
// and replace h[v] by the largest x <= h[v] such that at least x neighbours u
// have h[u] >= x.  Values only decrease and never fall below the core numbers;
// a sweep that changes nothing proves a fixed point, and a fixed point reached
// from above is the core numbers (if h[v] >= x, v has x neighbours with h >= x,
// so {h >= x} lies in the x-core).  Updates are in place (a neighbour's newer,
// smaller value only speeds convergence).  One wavefront per vertex.
// A sweep looks only at the vertices that the last one concerns (due[v] = its
// number; flag = kDue): a vertex whose value fell from a to b concerns itself and the
// neighbours with b < h <= a, of whose count it was one.  (A neighbour whose
// value fell in the same sweep, and may have been read before it did, concerns
// itself.)  After one that changed nothing the next looks at all (kAll), for rows
// that name each other need not be taken on trust, and if that changes nothing
// either, the values stand (kSettled).  A clique of true correspondences so is settled after two sweeps, and
// the rest of the graph after some more of about 6 us, the latencies of one row;
// re-reading all rows took 9 us a sweep (2,780 vertices, 2.8 million entries, 15
// sweeps; the first 104 us where a row's values were read again for each step of
// the search, now 20).  A row's loads are all in flight, and its values are searched in
// registers.  Six rounds per launch, each from a copy of h in LDS, took 60 us a
// launch: the copies of all blocks come from the same few lines.
enum : int { kSettled = 0, kAll = 1, kDue = 2 };  // what the next sweep is to do
constexpr int kHSweeps = 48;  // sweeps launched at most; the block peel finishes graphs that need more
constexpr int kHChunk = 8;    // sweeps between two looks of the host at the convergence flag
constexpr int kHRegs = 32;    // neighbour values held in registers per lane (deg <= 2048)
constexpr int kHFew = 4;      // and of short rows (deg <= 256): the checks of 32 were most of a sweep over them
                              // (16,000 vertices of 8 neighbours: 13 us a sweep, now 7)
static_assert(kHSweeps % kHChunk == 0, "whole chunks");

__global__ __launch_bounds__(kBlock) void kcore_hinit(const int32_t* __restrict__ off, int32_t n,
                                                      int32_t* __restrict__ h, int32_t* __restrict__ due,
                                                      int32_t* __restrict__ flag, int32_t* __restrict__ info) {
    if (blockIdx.x == 0 && threadIdx.x < 3) info[threadIdx.x] = 0;
    for (int v = blockIdx.x * kBlock + threadIdx.x; v < n; v += gridDim.x * kBlock) {
        h[v] = off[v + 1] - off[v];
        due[v] = 0;
    }
    for (int i = blockIdx.x * kBlock + threadIdx.x; i <= kHSweeps; i += gridDim.x * kBlock) flag[i] = i == 0 ? kAll : kSettled;
}

// The largest x <= hi that as many of a row's values reach, by their counts.
template <class F>
__device__ __forceinline__ int h_index(int hi, F count_ge) {
    int lo = count_ge(hi);
    if (lo >= hi) return hi;
    --hi;  // below hi as many values reach lo at least; count_ge(hi + 1) < hi + 1
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (count_ge(mid) >= mid) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// A row of at most 64 R neighbours (adj[b ..], deg of them) of vertex v, whose value
// is cap: its new value, and where that is less, the neighbours of whose count v was
// one are due.
template <int R>
__device__ __forceinline__ int sweep_row(const int32_t* __restrict__ adj, int32_t n, int32_t* h, int32_t* due, int v,
                                         int b, int deg, int cap, int next, int32_t* __restrict__ info) {
    const int lane = lane_id();
    int val[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int t = r * kWave + lane;
        val[r] = -1;
        if (r * kWave < deg) val[r] = t < deg ? adj[b + t] : -1;  // uniform
    }
    bool bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r * kWave >= deg) continue;  // uniform
        const int u = val[r];
        const bool in = u >= 0 && u < n;
        bad = bad || (!in && r * kWave + lane < deg);  // not a vertex: reported, never followed
        const int w = h[in ? u : v];
        val[r] = in ? w : -1;
    }
    if (bad) info[2] = 1;
    const int lo = h_index(min(cap, deg), [&](int x) {
        int c = 0;
#pragma unroll
        for (int r = 0; r < R; r += 4)
            if (r * kWave < deg)  // uniform
                c += __popcll(ballot(val[r] >= x)) + __popcll(ballot(val[r + 1] >= x)) +
                     __popcll(ballot(val[r + 2] >= x)) + __popcll(ballot(val[r + 3] >= x));
        return c;
    });
    if (lo < cap) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (r * kWave < deg && val[r] > lo && val[r] <= cap) due[adj[b + r * kWave + lane]] = next;
    }
    return lo;
}

__global__ __launch_bounds__(kBlock) void kcore_hsweep(const int32_t* __restrict__ off,
                                                       const int32_t* __restrict__ adj, int32_t n, int32_t* h, int32_t* due,
                                                       int32_t* flag, int sweep, int32_t* __restrict__ info) {
    const int lane = lane_id();
    const int todo = flag[sweep];
    bool changed = false;
    for (int64_t vw = global_wave(); vw < n; vw += wave_count()) {
        const int v = static_cast<int>(vw);
        const int now = due[v];
        const int cap = h[v];
        const int b = off[v], deg = off[v + 1] - b;
        if (todo == kSettled) return;  // looked at beside the row's own loads
        if (cap == 0 || (todo == kDue && now < sweep)) continue;
        int lo;
        if (deg <= kHFew * kWave) {  // uniform
            lo = sweep_row<kHFew>(adj, n, h, due, v, b, deg, cap, sweep + 1, info);
        } else if (deg <= kHRegs * kWave) {
            lo = sweep_row<kHRegs>(adj, n, h, due, v, b, deg, cap, sweep + 1, info);
        } else {  // re-read for each step of the search
            lo = h_index(min(cap, deg), [&](int x) {
                int c = 0;
                for (int t0 = 0; t0 < deg; t0 += kWave) {
                    const int t = t0 + lane;
                    int w = -1;
                    if (t < deg) {
                        const int u = adj[b + t];
                        if (u < 0 || u >= n) info[2] = 1;
                        else w = h[u];
                    }
                    c += __popcll(ballot(w >= x));
                }
                return c;
            });
            if (lo < cap)
                for (int t = lane; t < deg; t += kWave) {
                    const int u = adj[b + t];
                    if (u >= 0 && u < n && h[u] > lo && h[u] <= cap) due[u] = sweep + 1;
                }
        }
        if (lo < cap) {
            if (lane == 0) {
                h[v] = lo;
                due[v] = sweep + 1;
            }
            changed = true;
        }
    }
    if (changed && lane == 0) flag[sweep + 1] = kDue;
    if (todo == kDue && blockIdx.x == 0 && threadIdx.x == 0) atomicMax(flag + sweep + 1, static_cast<int>(kAll));
}

// One block: core numbers of the graph (off, adj) on n <= kMaxKcore vertices.
// Remaining degrees, core numbers and the list of the round's removals live in
// LDS (dynamic, 8 bytes per vertex), so the block's atomics and plain reads see
// one coherent copy.  A round removes every alive vertex whose remaining
// degree is <= the level (core number = level) and lists it; the block's
// wavefronts then take the listed vertices and their lanes walk each one's
// adjacency, decrementing alive neighbours.  A round that removes nothing
// raises the level to the smallest remaining degree (no round is spent on
// an empty level).
__global__ __launch_bounds__(kPeelThreads) void kcore_peel(const int32_t* __restrict__ off,
                                                           const int32_t* __restrict__ adj, int32_t n,
                                                           int32_t* __restrict__ core_out,
                                                           int32_t* __restrict__ info,
                                                           const int32_t* __restrict__ skip) {
    if (skip && *skip == kSettled) return;  // the h-index sweeps converged
    extern __shared__ int32_t s_mem[];
    int32_t* s_deg = s_mem;
    int16_t* s_core = reinterpret_cast<int16_t*>(s_deg + n);
    int16_t* s_list = s_core + n;
    __shared__ int s_cnt, s_left, s_min, s_max;
    const int lane = lane_id();
    const int wv = threadIdx.x / kWave;
    constexpr int kWaves = kPeelThreads / kWave;
    for (int v = threadIdx.x; v < n; v += kPeelThreads) {
        s_deg[v] = off[v + 1] - off[v];
        s_core[v] = -1;
    }
    if (threadIdx.x == 0) {
        s_left = n;
        s_max = -1;
    }
    int level = 0;
    while (true) {
        __syncthreads();
        if (s_left == 0) break;
        if (threadIdx.x == 0) {
            s_cnt = 0;
            s_min = INT_MAX;
        }
        __syncthreads();
        int low = INT_MAX;
        for (int v0 = 0; v0 < n; v0 += kPeelThreads) {
            const int v = v0 + threadIdx.x;
            bool rm = false;
            if (v < n && s_core[v] < 0) {
                const int d = s_deg[v];
                if (d <= level) {
                    s_core[v] = static_cast<int16_t>(level);
                    rm = true;
                } else {
                    low = min(low, d);
                }
            }
            const uint64_t b = ballot(rm);
            int base = 0;
            if (lane == 0 && b) base = atomicAdd(&s_cnt, __popcll(b));
            base = __shfl(base, 0, kWave);
            if (rm) s_list[base + lanes_below(b)] = static_cast<int16_t>(v);
        }
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) low = min(low, __shfl_xor(low, d, kWave));
        if (lane == 0 && low != INT_MAX) atomicMin(&s_min, low);
        __syncthreads();
        const int nrem = s_cnt;
        if (nrem == 0) {
            level = max(level + 1, s_min);  // every alive vertex has a larger degree
            continue;
        }
        if (threadIdx.x == 0) s_left -= nrem;
        for (int i = wv; i < nrem; i += kWaves) {
            const int f = s_list[i];
            const int e = off[f + 1];
            for (int t = off[f] + lane; t < e; t += kWave) {
                const int u = adj[t];
                if (u < 0 || u >= n) {  // not a vertex: reported, never followed
                    info[2] = 1;
                    continue;
                }
                if (s_core[u] < 0) atomicSub(&s_deg[u], 1);
            }
        }
    }
    int mx = -1;
    for (int v = threadIdx.x; v < n; v += kPeelThreads) {
        core_out[v] = s_core[v];
        mx = max(mx, static_cast<int>(s_core[v]));
    }
    atomicMax(&s_max, mx);
    __syncthreads();
    if (threadIdx.x == 0) info[0] = s_max;
}

size_t kcore_lds_bytes(int32_t n) { return static_cast<size_t>(n) * 8 + 16; }

// One block: core numbers (h, where the sweeps converged; else core and its
// maximum come from the peel) and members, the vertices with the largest core
// number, ascending.
__global__ __launch_bounds__(kPeelThreads) void kcore_members(const int32_t* __restrict__ h,
                                                              const int32_t* __restrict__ unsettled, int32_t* core,
                                                              int32_t n, int32_t* __restrict__ members,
                                                              int32_t* __restrict__ info) {
    __shared__ int s_base, s_max;
    __shared__ int s_wave[kPeelThreads / kWave];
    const int lane = lane_id();
    const int wv = threadIdx.x / kWave;
    const bool settled = *unsettled == kSettled;
    const int32_t* from = settled ? h : core;
    if (threadIdx.x == 0) {
        s_base = 0;
        s_max = settled ? -1 : info[0];
    }
    __syncthreads();
    if (settled) {
        int mx = -1;
        for (int v = threadIdx.x; v < n; v += kPeelThreads) {
            core[v] = h[v];
            mx = max(mx, h[v]);
        }
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) mx = max(mx, __shfl_xor(mx, d, kWave));
        if (lane == 0) atomicMax(&s_max, mx);
        __syncthreads();
    }
    const int mx = s_max;
    for (int v0 = 0; v0 < n; v0 += kPeelThreads) {
        const int v = v0 + threadIdx.x;
        const bool in = v < n && from[v] == mx;
        const uint64_t b = ballot(in);
        if (lane == 0) s_wave[wv] = __popcll(b);
        __syncthreads();
        int before = s_base;
        for (int w = 0; w < wv; ++w) before += s_wave[w];
        if (in) members[before + lanes_below(b)] = v;
        __syncthreads();
        if (threadIdx.x == 0) {
            int tot = 0;
            for (int w = 0; w < kPeelThreads / kWave; ++w) tot += s_wave[w];
            s_base += tot;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        info[0] = mx;
        info[1] = s_base;
    }
}

struct GraphWs {
    uint64_t* keys;
    int32_t* rank;
    float4* va;
    float4* vb;
    int32_t* deg;
    int64_t* nnz;
    int32_t* err;
    int64_t* scan_tmp;
};

GraphWs carve_graph(Carver& c, int64_t n_corr, int32_t n_tau) {
    GraphWs w;
    w.keys = c.take<uint64_t>(static_cast<size_t>(std::max<int64_t>(n_corr, 1)));
    w.rank = c.take<int32_t>(static_cast<size_t>(std::max<int64_t>(n_corr, 1)));
    w.va = c.take<float4>(static_cast<size_t>(std::max(n_tau, 1)));
    w.vb = c.take<float4>(static_cast<size_t>(std::max(n_tau, 1)));
    w.deg = c.take<int32_t>(static_cast<size_t>(n_tau) + 1);
    w.nnz = c.take<int64_t>(1);
    w.err = c.take<int32_t>(2);  // an index outside its cloud; a bounded wait that gave up
    w.scan_tmp = c.take<int64_t>(scan_temp_elems(static_cast<int64_t>(n_tau) + 1));
    return w;
}

struct KcoreWs {
    int32_t* info;
    int32_t* h;
    int32_t* due;
    int32_t* flag;
};

KcoreWs carve_kcore(Carver& c, int32_t n) {
    KcoreWs w;
    w.info = c.take<int32_t>(3);  // max core, members, bad index flag
    w.h = c.take<int32_t>(static_cast<size_t>(std::max(n, 1)));
    w.due = c.take<int32_t>(static_cast<size_t>(std::max(n, 1)));
    w.flag = c.take<int32_t>(kHSweeps + 1);
    return w;
}

}  // namespace

size_t graph_ws(int64_t n_corr, int32_t n_tau) {
    Carver c(nullptr, 0);
    carve_graph(c, n_corr, n_tau);
    return c.off;
}

size_t kcore_ws(int32_t n) {
    Carver c(nullptr, 0);
    carve_kcore(c, n);
    return c.off;
}

kmg_status corr_graph(const float* src, int64_t src_stride, const float* tgt, int64_t tgt_stride,
                      const int32_t* pairs, const float* d1, const float* d2, int64_t n_corr, int32_t n_tau,
                      double beta, int32_t* sel, int32_t* off, int32_t* adj, int64_t adj_cap, int32_t* n_sel_host,
                      int64_t* nnz_host, void* ws, size_t ws_bytes, hipStream_t s) {
    Carver c(ws, ws_bytes);
    GraphWs w = carve_graph(c, n_corr, n_tau);
    if (!c.fits()) return KMG_ERR_WORKSPACE;
    const int32_t n = static_cast<int32_t>(std::min<int64_t>(n_corr, n_tau));
    *n_sel_host = n;
    *nnz_host = 0;
    if (n == 0) {
        KMG_TRY(fill_u32(reinterpret_cast<uint32_t*>(off), 0u, 1, s));
        return KMG_OK;
    }
    FillJobs fills{};
    fills.job[0] = FillJob{w.err, 0ull, 2, 4};
    fills.job[1] = FillJob{w.deg, 0ull, static_cast<int64_t>(n) + 1, 4};
    fills.job[2] = FillJob{w.scan_tmp, 0ull, static_cast<int64_t>(scan_temp_elems(static_cast<int64_t>(n) + 1)), 8};
    fills.n_jobs = 3;
    ratio_keys<<<grid_cap(n_corr, kBlock), kBlock, 0, s>>>(d1, d2, n_corr, w.keys, w.rank, fills);
    KMG_TRY(launch_status());
    {
        const int64_t tiles = (n_corr + kBlock - 1) / kBlock;
        const dim3 grid(static_cast<unsigned>(tiles), static_cast<unsigned>(std::min<int64_t>(tiles, kRankTiles)));
        rank_count<<<grid, kBlock, 0, s>>>(w.keys, n_corr, w.rank);
        KMG_TRY(launch_status());
    }
    gather_vertices<<<grid_cap(n_corr, kBlock), kBlock, 0, s>>>(src, src_stride, tgt, tgt_stride, pairs, w.rank,
                                                                n_corr, n_tau, sel, w.va, w.vb, w.err);
    KMG_TRY(launch_status());
    graph_rows<false><<<grid_cap(n, kBlock / kWave), kBlock, 0, s>>>(w.va, w.vb, n, beta, w.deg, nullptr, nullptr);
    KMG_TRY(launch_status());
    KMG_TRY(scan_exclusive_onepass(w.deg, off, static_cast<int64_t>(n) + 1, w.nnz,
                                   reinterpret_cast<uint64_t*>(w.scan_tmp), w.err + 1, s));
    int64_t nnz = 0;
    int32_t err[2] = {0, 0};
    Report r;
    KMG_TRY(r.post(w.nnz, sizeof(nnz), w.err, sizeof(err), s));
    KMG_TRY(r.wait(&nnz, err));
    if (err[0]) return KMG_ERR_RANGE;
    if (err[1]) return KMG_ERR_DEVICE;
    *nnz_host = nnz;
    if (nnz > adj_cap) return KMG_ERR_CAPACITY;
    graph_rows<true><<<grid_cap(n, kBlock / kWave), kBlock, 0, s>>>(w.va, w.vb, n, beta, nullptr, off, adj);
    KMG_TRY(launch_status());
    return KMG_OK;
}

kmg_status max_kcore(const int32_t* off, const int32_t* adj, int32_t n, int32_t* core, int32_t* members,
                     int32_t* n_members_host, int32_t* max_core_host, void* ws, size_t ws_bytes, hipStream_t s) {
    Carver c(ws, ws_bytes);
    KcoreWs w = carve_kcore(c, n);
    if (!c.fits()) return KMG_ERR_WORKSPACE;
    *n_members_host = 0;
    *max_core_host = -1;
    if (n == 0) return KMG_OK;
    const size_t lds = kcore_lds_bytes(n);
    if (lds > 65536) {
        static const hipError_t raised = hipFuncSetAttribute(reinterpret_cast<const void*>(&kcore_peel),
                                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                                             static_cast<int>(kcore_lds_bytes(kMaxKcore)));
        if (raised != hipSuccess) return KMG_ERR_RANGE;  // this device cannot hold the graph's state on chip
    }
    kcore_hinit<<<grid_cap(std::max<int64_t>(n, kHSweeps + 1), kBlock), kBlock, 0, s>>>(off, n, w.h, w.due, w.flag, w.info);
    KMG_TRY(launch_status());
    // Sweeps in chunks, one chunk ahead of the host's look at the flag: launches past convergence
    // do nothing, but cost 2 us each (26 of the 48 for 2,780 vertices).
    Report seen[2];
    bool settled = false;
    for (int k = 0, chunk = 0; k < kHSweeps && !settled; ++chunk) {
        for (const int end = k + kHChunk; k < end; ++k) {
            kcore_hsweep<<<grid_cap(n, kBlock / kWave), kBlock, 0, s>>>(off, adj, n, w.h, w.due, w.flag, k, w.info);
            KMG_TRY(launch_status());
        }
        KMG_TRY(seen[chunk & 1].post(w.flag + k, sizeof(int32_t), nullptr, 0, s));
        int32_t more = kDue;
        if (chunk > 0) KMG_TRY(seen[(chunk - 1) & 1].wait(&more));
        settled = more == kSettled;
    }
    if (!settled) {
        kcore_peel<<<1, kPeelThreads, lds, s>>>(off, adj, n, core, w.info, w.flag + kHSweeps);
        KMG_TRY(launch_status());
    }
    kcore_members<<<1, kPeelThreads, 0, s>>>(w.h, w.flag + kHSweeps, core, n, members, w.info);
    KMG_TRY(launch_status());
    int32_t info[3];
    Report r;
    KMG_TRY(r.post(w.info, sizeof(info), nullptr, 0, s));
    KMG_TRY(r.wait(info));
    int32_t last = 0;
    for (Report& q : seen)
        if (q.posted()) KMG_TRY(q.wait(&last));  // here already
    if (info[2]) return KMG_ERR_RANGE;
    *max_core_host = info[0];
    *n_members_host = info[1];
    return KMG_OK;
}

}  // namespace kmg
