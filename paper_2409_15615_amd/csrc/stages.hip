// Single-cloud entry points: batches of one cloud run through the batch
// kernels, with the counts brought back to the host at the end of each call.
#include "kmg_device.h"

namespace kmg {

namespace {

// Clears the status, writes the cloud's record (block 0) and does the fills of
// the call (a launch each, they were half of a small call's launches).
// off (optional): the caller's neighbour lists, whose volume off[m_kept] goes
// to st->nnz.  r (optional): the points' records from the caller's arrays.
struct RecJob {
    float4* rec;
    const float* xyz;
    const float* nrm;
    const uint8_t* flags;
};
__global__ __launch_bounds__(256) void init_single(DevStatus* st, CloudDev* cl, CloudDev v, int64_t n_raw,
                                                   int64_t m_kept, const int32_t* off, FillJobs fills, RecJob r) {
    if (blockIdx.x == 0) {
        const int i = threadIdx.x;
        uint32_t* w = reinterpret_cast<uint32_t*>(st);
        for (int k = i; k < static_cast<int>(sizeof(DevStatus) / 4); k += blockDim.x) w[k] = 0u;
        __syncthreads();
        if (i == 0) {
            st->n_raw = n_raw;
            st->m_kept = m_kept;
            if (off) st->nnz = off[m_kept];
            cl[0] = v;
        }
    }
    run_fill_jobs(fills);
    if (!r.rec) return;
    for (int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; q < m_kept;
         q += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        r.rec[2 * q] = make_float4(r.xyz[q], r.xyz[m_kept + q], r.xyz[2 * m_kept + q], __int_as_float(r.flags[q] & 1));
        r.rec[2 * q + 1] = make_float4(r.nrm[q], r.nrm[m_kept + q], r.nrm[2 * m_kept + q], 0.f);
    }
}

void add_fill(FillJobs& f, void* p, uint64_t v, int64_t n, int32_t bytes) { f.job[f.n_jobs++] = FillJob{p, v, n, bytes}; }

// The cell hash, the degrees and the look-back words of a search over m points.
void add_search_fills(FillJobs& f, const SearchWs& w, int64_t m) {
    add_fill(f, w.keys, kEmptyKey, w.cap_table, 8);
    add_fill(f, w.ccount, 0ull, w.cap_table, 4);
    add_fill(f, w.cfill, 0ull, w.cap_table, 4);
    add_fill(f, w.deg, 0ull, m + 1, 4);
    add_fill(f, w.scan_tmp, 0ull, static_cast<int64_t>(search_scan_status_elems(w, m)), 8);
}

kmg_status init(DevStatus* st, CloudDev* cl, const CloudDev& v, int64_t n_raw, int64_t m_kept, const FillJobs& fills,
                hipStream_t s, const int32_t* off = nullptr, const RecJob& r = RecJob{}) {
    int64_t most = std::max<int64_t>(r.rec ? m_kept : 1, 1);
    for (int k = 0; k < fills.n_jobs; ++k) most = std::max(most, fills.job[k].n);
    init_single<<<static_cast<unsigned>(std::min<int64_t>((most + 255) / 256, 4096)), 256, 0, s>>>(st, cl, v, n_raw,
                                                                                                  m_kept, off, fills, r);
    return launch_status();
}

uint64_t* look_back_words(int64_t* scan_tmp) { return reinterpret_cast<uint64_t*>(scan_tmp); }

kmg_status read_status(DevStatus* st, DevStatus* host, hipStream_t s) {
    Report r;
    KMG_TRY(r.post(st, sizeof(DevStatus), nullptr, 0, s));
    KMG_TRY(r.wait(host));
    timer_collect();
    return KMG_OK;
}

// The fill after a count pass.  The lists go first, behind the report of the
// count: while the host reads it the GPU already fills (nothing, when the lists
// exceed the capacity, their offsets or the supported range).  A call that is refused
// waits for that launch, which reads the workspace: the caller may use or free it next.
kmg_status fill_counted(const CloudDev* cl, const float* xyz, int64_t m, int64_t nbr_cap, DevStatus* st,
                        const SearchWs& w, const int32_t* off, int32_t* nbr, float* nrm, uint8_t* flags,
                        int32_t* n_normal, hipStream_t s, int use_rn, bool with_normals, int64_t* nnz_host,
                        kmg_status over_capacity) {
    Report r;
    DevStatus h;
    const int64_t cap = std::min<int64_t>(nbr_cap, INT32_MAX);  // 32-bit offsets
    KMG_TRY(r.post(st, sizeof(DevStatus), nullptr, 0, s));
    KMG_TRY(search_fill_batch(cl, xyz, m, nullptr, m, cap, kFillLists, st, w, off, nbr, nrm, m, flags, n_normal, s,
                              use_rn));
    KMG_TRY(r.wait(&h));
    timer_collect();
    kmg_status refused = KMG_OK;
    if (h.err_sync) {
        refused = KMG_ERR_DEVICE;
    } else if (h.err_range || (h.dense & 2) || h.nnz > INT32_MAX) {
        refused = KMG_ERR_RANGE;
    } else {
        if (nnz_host) *nnz_host = h.nnz;
        if (h.nnz > nbr_cap) refused = over_capacity;
    }
    if (refused != KMG_OK) {
        KMG_TRY_HIP(hipStreamSynchronize(s));
        return refused;
    }
    return search_fill_batch(cl, xyz, m, nullptr, m, cap,
                             ((h.dense & 1) ? kFillDense : 0) | (with_normals ? kFillNormals : 0), st, w, off, nbr, nrm,
                             m, flags, n_normal, s, use_rn);
}

}  // namespace

CloudDev make_cloud(const kmg_params& p, const float* raw, int64_t n_raw, int64_t raw_off) {
    CloudDev c{};
    c.raw = raw;
    c.n_raw = static_cast<int32_t>(n_raw);
    c.raw_off = static_cast<int32_t>(raw_off);
    c.tau_num = p.tau_num;
    c.H = p.n_bins;
    c.voxel = p.voxel;
    c.inv_cell = 1.0 / (p.r_fpfh * (1.0 + 1e-4));
    c.tau_lin = p.tau_lin;
    for (int k = 0; k < 3; ++k) c.vp[k] = p.viewpoint[k];
    c.rf = make_radius_test(p.r_fpfh);
    c.rn = make_radius_test(p.r_normal);
    c.mode = p.mode;
    c.tau_j = p.tau_num;
    if (p.mode == KMG_MODE_CLASSIC_FPFH) {
        // classic FPFH: a normal for any point with >= 3 r_normal neighbours, no
        // linearity filter, a descriptor for every point with a normal
        c.tau_num = 3;
        c.tau_lin = 1.0;
        c.tau_j = 1;
    }
    return c;
}

size_t voxelize_ws(int64_t n) {
    Carver c(nullptr, 0);
    c.take<DevStatus>(1);
    c.take<CloudDev>(1);
    carve_voxel(c, n);
    return c.off;
}

kmg_status voxelize(const float* xyz, int64_t n, double voxel, int32_t* kept_idx, float* kept_xyz, int64_t cap,
                    int64_t* n_kept_host, void* ws, size_t ws_bytes, hipStream_t s) {
    Carver c(ws, ws_bytes);
    DevStatus* st = c.take<DevStatus>(1);
    CloudDev* cl = c.take<CloudDev>(1);
    VoxelWs w = carve_voxel(c, n);
    if (!c.fits()) return KMG_ERR_WORKSPACE;
    kmg_params p{};
    p.voxel = voxel;
    p.r_normal = p.r_fpfh = voxel;
    p.tau_lin = 1.0;
    p.tau_num = 1;
    p.n_bins = 1;
    FillJobs fills{};
    add_fill(fills, w.keys, kEmptyKey, w.cap_table, 8);
    add_fill(fills, w.mins, 0x7fffffffull, w.cap_table, 4);
    add_fill(fills, w.scan_tmp, 0ull, static_cast<int64_t>(scan_temp_elems(n)), 8);
    KMG_TRY(init(st, cl, make_cloud(p, xyz, n, 0), n, 0, fills, s));
    KMG_TRY(voxelize_batch(cl, 1, n, st, w, cap, 0, kept_idx, kept_xyz, nullptr, nullptr, s, true, nullptr,
                           look_back_words(w.scan_tmp)));
    DevStatus h;
    KMG_TRY(read_status(st, &h, s));
    if (h.err_range) return KMG_ERR_RANGE;
    if (h.err_sync) return KMG_ERR_DEVICE;
    *n_kept_host = h.m_kept;
    if (h.m_kept > cap) return KMG_ERR_CAPACITY;
    return KMG_OK;
}

size_t normals_ws(int64_t m, int mode, int64_t nbr_cap) {
    Carver c(nullptr, 0);
    c.take<DevStatus>(1);
    c.take<CloudDev>(1);
    carve_search(c, m);
    if (mode == KMG_MODE_CLASSIC_FPFH) {  // the separate r_normal lists
        c.take<int32_t>(static_cast<size_t>(m) + 1);
        c.take<int32_t>(static_cast<size_t>(std::max<int64_t>(nbr_cap, 1)));
    }
    return c.off;
}

kmg_status normals(const float* xyz, int64_t m, const kmg_params& p, float* nrm, uint8_t* flags, int32_t* off,
                   int32_t* nbr, int64_t nbr_cap, int64_t* nnz_host, int32_t* n_normal, void* ws, size_t ws_bytes,
                   hipStream_t s) {
    Carver c(ws, ws_bytes);
    DevStatus* st = c.take<DevStatus>(1);
    CloudDev* cl = c.take<CloudDev>(1);
    SearchWs w = carve_search(c, m);
    const bool classic = p.mode == KMG_MODE_CLASSIC_FPFH;
    int32_t* off_n = nullptr;
    int32_t* nbr_n = nullptr;
    int64_t nbr_n_cap = 0;
    if (classic) {
        off_n = c.take<int32_t>(static_cast<size_t>(m) + 1);
        nbr_n_cap = std::max<int64_t>(nbr_cap, 1);
        nbr_n = c.take<int32_t>(static_cast<size_t>(nbr_n_cap));
    }
    if (!c.fits()) return KMG_ERR_WORKSPACE;
    FillJobs fills{};
    add_search_fills(fills, w, m);
    KMG_TRY(init(st, cl, make_cloud(p, nullptr, 0, 0), 0, m, fills, s));
    if (classic) {
        // search 1 (r_normal) and the normals from its lists
        KMG_TRY(search_count_batch(cl, xyz, m, nullptr, m, st, w, off_n, s, true, 1, true, false,
                                   look_back_words(w.scan_tmp)));
        int64_t nnz_n = 0;
        const kmg_status got = fill_counted(cl, xyz, m, nbr_n_cap, st, w, off_n, nbr_n, nrm, flags, n_normal, s, 1,
                                            true, &nnz_n, KMG_ERR_CAPACITY);
        if (got == KMG_ERR_CAPACITY) *nnz_host = nnz_n;
        KMG_TRY(got);
    }
    // Faster-PFH: the one search at r_FPFH; classic: search 2, lists only, over the same grid
    if (classic)
        KMG_TRY(search_count_batch(cl, xyz, m, nullptr, m, st, w, off, s, false, 0));
    else
        KMG_TRY(search_count_batch(cl, xyz, m, nullptr, m, st, w, off, s, true, 0, true, false,
                                   look_back_words(w.scan_tmp)));
    KMG_TRY(fill_counted(cl, xyz, m, nbr_cap, st, w, off, nbr, nrm, flags, n_normal, s, 0, !classic, nnz_host,
                         KMG_ERR_CAPACITY));
    timer_collect();
    return KMG_OK;
}

size_t fpfh_ws(int64_t m, int H, int mode, int64_t nnz) {
    Carver c(nullptr, 0);
    c.take<DevStatus>(1);
    c.take<CloudDev>(1);
    carve_feat(c, m, H);
    if (mode == KMG_MODE_CLASSIC_FPFH) {  // search 3: its own grid and lists
        carve_search(c, m);
        c.take<int32_t>(static_cast<size_t>(m) + 1);
        c.take<int32_t>(static_cast<size_t>(std::max<int64_t>(nnz, 1)));
    }
    return c.off;
}

kmg_status fpfh(const float* xyz, const float* nrm, uint8_t* flags, const int32_t* off, const int32_t* nbr,
                int64_t m, const kmg_params& p, float* spfh_out, float* fpfh_out, int32_t* j_idx, int64_t* n_j_host,
                int64_t* stats_host, void* ws, size_t ws_bytes, hipStream_t s) {
    const int H = p.n_bins;
    Carver c(ws, ws_bytes);
    DevStatus* st = c.take<DevStatus>(1);
    CloudDev* cl = c.take<CloudDev>(1);
    FeatWs w = carve_feat(c, m, H);
    const bool classic = p.mode == KMG_MODE_CLASSIC_FPFH;
    SearchWs sw{};
    int32_t* off3 = nullptr;
    int32_t* nbr3 = nullptr;
    int64_t nnz3_cap = 0;
    if (classic) {
        sw = carve_search(c, m);
        off3 = c.take<int32_t>(static_cast<size_t>(m) + 1);
        // the rest of the workspace holds search 3's lists (less the carver's alignment)
        nnz3_cap = static_cast<int64_t>((ws_bytes > c.off + 512 ? ws_bytes - c.off - 512 : 0) / sizeof(int32_t));
        nbr3 = c.take<int32_t>(static_cast<size_t>(std::max<int64_t>(nnz3_cap, 1)));
    }
    if (!c.fits()) return KMG_ERR_WORKSPACE;
    FillJobs fills{};
    add_fill(fills, w.jflag, 0ull, std::max<int64_t>(m, 1), 4);
    add_fill(fills, w.scan_tmp, 0ull, static_cast<int64_t>(scan_temp_elems(m)), 8);
    if (classic) add_search_fills(fills, sw, m);
    KMG_TRY(init(st, cl, make_cloud(p, nullptr, 0, 0), 0, m, fills, s, off, RecJob{w.rec, xyz, nrm, flags}));
    if (!classic) {
        KMG_TRY(features_batch(cl, 1, xyz, m, nullptr, m, H, st, w, off, NbrLists{nbr}, flags, spfh_out,
                               fpfh_out, j_idx, nullptr, s, true, nullptr, look_back_words(w.scan_tmp)));
    } else {
        // SPFH over the lists of search 2; search 3 (r_FPFH again) for the FPFH sum
        KMG_TRY(spfh_batch(cl, nullptr, m, H, st, w, off, NbrLists{nbr}, spfh_out, s, true));
        KMG_TRY(search_count_batch(cl, xyz, m, nullptr, m, st, sw, off3, s, true, 0, true, false,
                                   look_back_words(sw.scan_tmp)));
        KMG_TRY(fill_counted(cl, xyz, m, nnz3_cap, st, sw, off3, nbr3, nullptr, flags, nullptr, s, 0, false, nullptr,
                             KMG_ERR_WORKSPACE));
        KMG_TRY(fpfh_batch(1, xyz, m, m, H, st, w, off3, NbrLists{nbr3}, flags, fpfh_out, j_idx, nullptr, s, nullptr,
                           look_back_words(w.scan_tmp)));
    }
    DevStatus h;
    KMG_TRY(read_status(st, &h, s));
    if (h.err_sync) return KMG_ERR_DEVICE;
    *n_j_host = h.n_j;
    if (stats_host) {
        stats_host[0] = h.feat_fp64;
        stats_host[1] = h.feat_edge;
    }
    return KMG_OK;
}

}  // namespace kmg
