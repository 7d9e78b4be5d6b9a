// Small transfers between host and device.
//
// A read of a few hundred bytes (a box's state, two energies, one move's
// results) is bound by the latency of the way it takes, not by its bytes.  As a
// copy into pageable memory and a stream synchronisation it took 20.7 us, with
// pinned memory 11.2 us; here a kernel behind the stream's work writes the words
// and then a ticket to a slot of pinned memory, which the host polls: 6.7 us.  A
// write of up to kWriteBytes travels in a kernel's arguments, which the launch
// copies: 2.5 us and no wait, where the copy took 12.3 us.  Larger transfers are
// bound by the copy itself and are left to it.
#include <string.h>

#include <chrono>
#include <mutex>

#include "gcmc_internal.h"

namespace gcmc {

constexpr int kReadSlots = 16;       // reads in flight at once; a further one takes the copy
constexpr int kReadWords = 1024;     // 4 KB a slot: the copy's rate wins from about there
constexpr int kWriteBytes = 2048;    // half of the space a launch has for arguments
constexpr int kPollMicros = 500;     // then the stream is waited for instead

struct ReadSlot {
    uint32_t ticket;                 // of the read whose words are here, in a cache line of its own
    uint32_t pad[15];
    uint32_t w[kReadWords];
};
struct WriteWords {
    uint32_t w[kWriteBytes / 4];
};

__global__ __launch_bounds__(256) void k_publish(const uint32_t* __restrict__ src, int words, ReadSlot* slot,
                                                 uint32_t ticket) {
    for (int i = threadIdx.x; i < words; i += blockDim.x) slot->w[i] = src[i];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&slot->ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void k_write_words(WriteWords v, uint32_t* dst, int words) {
    for (int i = threadIdx.x; i < words; i += blockDim.x) dst[i] = v.w[i];
}

namespace {

// The slots: one pinned allocation, made with the first box (not by a read, which
// another stream's capture could forbid it) and given back when the last box is gone.  A slot is one call's from take to give; the lock is not held
// while a call waits.
class ReadSlots {
  public:
    void retain() {
        std::lock_guard<std::mutex> g(mu_);
        ++users_;
        if (base_) return;
        void* p = nullptr;
        if (hipHostMalloc(&p, sizeof(ReadSlot) * kReadSlots, hipHostMallocPortable | hipHostMallocCoherent) !=
            hipSuccess) {
            (void)hipGetLastError();   // reads take the copy
            return;
        }
        base_ = static_cast<ReadSlot*>(p);
        memset(p, 0, sizeof(ReadSlot) * kReadSlots);
        for (int k = 0; k < kReadSlots; ++k) next_[k] = 0;
    }
    void release() {
        std::lock_guard<std::mutex> g(mu_);
        --users_;
        drop_unused();
    }
    int take(ReadSlot** slot, uint32_t* ticket) {
        std::lock_guard<std::mutex> g(mu_);
        if (users_ <= 0 || !base_) return -1;
        for (int k = 0; k < kReadSlots; ++k)
            if (!(used_ >> k & 1)) {
                used_ |= 1u << k;
                *slot = base_ + k;
                *ticket = ++next_[k] ? next_[k] : ++next_[k];   // 0 is no ticket
                return k;
            }
        return -1;
    }
    void give(int k) {
        std::lock_guard<std::mutex> g(mu_);
        used_ &= ~(1u << k);
        drop_unused();
    }

  private:
    void drop_unused() {
        if (users_ > 0 || used_ != 0 || !base_) return;
        (void)hipHostFree(base_);
        base_ = nullptr;
    }
    std::mutex mu_;
    ReadSlot* base_ = nullptr;
    int users_ = 0;
    uint32_t used_ = 0;
    uint32_t next_[kReadSlots] = {0};
};

ReadSlots& slots() {
    static ReadSlots* s = new ReadSlots();   // never destroyed: boxes may outlive static objects
    return *s;
}

int read_by_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
    GCMC_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s));
    GCMC_HIP(hipStreamSynchronize(s));
    return GCMC_OK;
}

}  // namespace

// A capturing stream (or a capture that forbids work on this one) goes to the copy,
// which reports it as it always did.
bool stream_capturing(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

void transfer_retain() { slots().retain(); }
void transfer_release() { slots().release(); }

int read_back(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (bytes == 0) return GCMC_OK;
    if (bytes > 4 * kReadWords || bytes % 4 != 0 || (uintptr_t)src % 4 != 0 || stream_capturing(s))
        return read_by_copy(dst, src, bytes, s);
    ReadSlot* slot = nullptr;
    uint32_t ticket = 0;
    const int k = slots().take(&slot, &ticket);
    if (k < 0) return read_by_copy(dst, src, bytes, s);
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(256), 0, s, (const uint32_t*)src, (int)(bytes / 4), slot, ticket);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {   // nothing was launched
        slots().give(k);
        return check_hip(e, "read_back");
    }
    const auto t0 = std::chrono::steady_clock::now();
    bool there = false;
    do {
        for (int i = 0; i < 64 && !there; ++i) there = __atomic_load_n(&slot->ticket, __ATOMIC_ACQUIRE) == ticket;
    } while (!there && std::chrono::steady_clock::now() - t0 < std::chrono::microseconds(kPollMicros));
    if (!there) {
        e = hipStreamSynchronize(s);
        there = __atomic_load_n(&slot->ticket, __ATOMIC_ACQUIRE) == ticket;
        // a slot that the device may still write to is not used again
        if (e != hipSuccess) return check_hip(e, "hipStreamSynchronize(s)");
        if (!there) return set_error(GCMC_ERR_HIP, "a read behind the stream's work did not arrive");
    }
    memcpy(dst, slot->w, bytes);
    slots().give(k);
    return GCMC_OK;
}

}  // namespace gcmc

using namespace gcmc;

extern "C" {

int gcmc_read(void* h_dst, const void* d_src, int64_t bytes, void* stream) {
    if (bytes < 0 || (bytes > 0 && (!h_dst || !d_src))) return set_error(GCMC_ERR_INVALID_ARG, "bad arguments");
    return read_back(h_dst, d_src, (size_t)bytes, (hipStream_t)stream);
}

int gcmc_write(void* d_dst, const void* h_src, int64_t bytes, void* stream) {
    if (bytes < 0 || (bytes > 0 && (!d_dst || !h_src))) return set_error(GCMC_ERR_INVALID_ARG, "bad arguments");
    if (bytes == 0) return GCMC_OK;
    hipStream_t s = (hipStream_t)stream;
    if (bytes > kWriteBytes || bytes % 4 != 0 || (uintptr_t)d_dst % 4 != 0 || stream_capturing(s)) {
        GCMC_HIP(hipMemcpyAsync(d_dst, h_src, (size_t)bytes, hipMemcpyHostToDevice, s));
        GCMC_HIP(hipStreamSynchronize(s));
        return GCMC_OK;
    }
    WriteWords v;
    memcpy(v.w, h_src, (size_t)bytes);
    hipLaunchKernelGGL(k_write_words, dim3(1), dim3(256), 0, s, v, (uint32_t*)d_dst, (int)(bytes / 4));
    GCMC_HIP(hipGetLastError());
    return GCMC_OK;
}

}  // extern "C"
