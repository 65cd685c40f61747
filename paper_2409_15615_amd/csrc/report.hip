// Brings a call's few result words back to the host.
//
// A copy into pageable memory is a staging kernel, a host copy and a wait for
// the stream's completion signal: about 30 us from the end of the last kernel
// to the return of the call.  Here a one-wavefront kernel at that point of the
// stream writes the words into pinned host memory and then a ticket, which the
// host polls: about 8 us.  A wait that takes long gives way to the stream's own
// synchronisation, which also reports what went wrong.
//
// The pinned slots come from a pool shared by all threads (a slot belongs to one
// call at a time); at most kPoolSlots of them are kept.
#include <sched.h>
#include <string.h>

#include <chrono>
#include <mutex>

#include "kmg_device.h"

namespace kmg {

namespace {

constexpr int kPoolSlots = 16;
constexpr auto kYieldAfter = std::chrono::microseconds(100);
constexpr auto kSyncAfter = std::chrono::milliseconds(2);

__global__ __launch_bounds__(kWave) void report_words(const uint32_t* a, int na, const uint32_t* b, int nb,
                                                      ReportSlot* out, uint32_t ticket) {
    for (int k = threadIdx.x; k < na; k += kWave) out->words[k] = a[k];
    for (int k = threadIdx.x; k < nb; k += kWave) out->words[na + k] = b[k];
    __threadfence_system();  // every lane's words are out before the ticket (one wavefront)
    if (threadIdx.x == 0) __hip_atomic_store(&out->ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

std::mutex g_mu;
ReportSlot* g_free[kPoolSlots];
int g_n_free = 0;

}  // namespace

Report::~Report() {
    if (!slot_) return;
    if (posted_) return;  // a kernel may still write the slot: it is not used again
    {
        std::lock_guard<std::mutex> lock(g_mu);
        if (g_n_free < kPoolSlots) {
            g_free[g_n_free++] = slot_;
            return;
        }
    }
    (void)hipHostFree(slot_);
}

kmg_status Report::post(const void* a, size_t a_bytes, const void* b, size_t b_bytes, hipStream_t s) {
    const int na = static_cast<int>(a_bytes / 4), nb = static_cast<int>(b_bytes / 4);
    if (na + nb > kReportWords || posted_) return KMG_ERR_ARG;
    if (!slot_) {
        {
            std::lock_guard<std::mutex> lock(g_mu);
            if (g_n_free > 0) slot_ = g_free[--g_n_free];
        }
        if (!slot_) {
            void* p = nullptr;
            if (hipHostMalloc(&p, sizeof(ReportSlot), hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) {
                slot_ = static_cast<ReportSlot*>(p);
                slot_->ticket = 0;
            } else {
                (void)hipGetLastError();  // no pinned memory to be had: wait() copies
            }
        }
    }
    na_ = na;
    nb_ = nb;
    stream_ = s;
    a_ = a;
    b_ = b;
    if (!slot_) {
        posted_ = true;
        return KMG_OK;
    }
    void* dev = nullptr;
    KMG_TRY_HIP(hipHostGetDevicePointer(&dev, slot_, 0));
    ticket_ = slot_->ticket + 1;
    report_words<<<1, kWave, 0, s>>>(static_cast<const uint32_t*>(a), na, static_cast<const uint32_t*>(b), nb,
                                     static_cast<ReportSlot*>(dev), ticket_);
    KMG_TRY(launch_status());
    posted_ = true;
    return KMG_OK;
}

kmg_status Report::wait(void* a, void* b) {
    if (!posted_) return KMG_ERR_ARG;
    if (!slot_) {
        posted_ = false;
        KMG_TRY_HIP(hipMemcpyAsync(a, a_, static_cast<size_t>(na_) * 4, hipMemcpyDeviceToHost, stream_));
        if (nb_) KMG_TRY_HIP(hipMemcpyAsync(b, b_, static_cast<size_t>(nb_) * 4, hipMemcpyDeviceToHost, stream_));
        KMG_TRY_HIP(hipStreamSynchronize(stream_));
        return KMG_OK;
    }
    const auto there = [&] { return __atomic_load_n(&slot_->ticket, __ATOMIC_ACQUIRE) == ticket_; };
    const auto t0 = std::chrono::steady_clock::now();
    while (!there()) {
        for (int k = 0; k < 32 && !there(); ++k) __builtin_ia32_pause();
        const auto waited = std::chrono::steady_clock::now() - t0;
        if (waited > kSyncAfter) {
            KMG_TRY_HIP(hipStreamSynchronize(stream_));
            if (!there()) return KMG_ERR_DEVICE;
        } else if (waited > kYieldAfter) {
            sched_yield();
        }
    }
    posted_ = false;
    memcpy(a, slot_->words, static_cast<size_t>(na_) * 4);
    if (nb_) memcpy(b, slot_->words + na_, static_cast<size_t>(nb_) * 4);
    return KMG_OK;
}

}  // namespace kmg
