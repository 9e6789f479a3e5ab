// Eight words of page-locked host memory for what one build has to know from its kernels (host code only).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <mutex>

// The fold kernel writes the words itself, so that planning the sort waits for a kernel and not for a copy behind
// it. 64 builds of the process can hold eight words at a time (a page that stays until it ends); a further one finds
// `words` null and reads its result back from the scratch block instead.
//
// A slot goes to another build only once nothing can write it any more: launched() says that kernels which may
// are on their way, settled() that their stream has been waited for. Where an error came between the two the
// destructor waits; if even that fails (a broken device, a stream under capture) the slot is never used again.
struct PinnedInfo {
    unsigned long long* words = nullptr;
    PinnedInfo() {
        std::lock_guard<std::mutex> lock(mutex());
        State& s = state();
        if (!s.page && !s.failed) {
            void* p = nullptr;
            if (hipHostMalloc(&p, 64 * 64, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) s.page = static_cast<uint8_t*>(p);
            else {
                s.failed = true;
                (void)hipGetLastError();
            }
        }
        if (s.page && ~s.used) {
            slot_ = __builtin_ctzll(~s.used);
            s.used |= 1ull << slot_;
            words = reinterpret_cast<unsigned long long*>(s.page + 64 * slot_);
        }
    }
    ~PinnedInfo() {
        if (!words) return;
        if (pending_ && hipStreamSynchronize(stream_) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        std::lock_guard<std::mutex> lock(mutex());
        state().used &= ~(1ull << slot_);
    }
    PinnedInfo(const PinnedInfo&) = delete;
    PinnedInfo& operator=(const PinnedInfo&) = delete;
    void launched(hipStream_t stream) {
        stream_ = stream;
        pending_ = true;
    }
    void settled() { pending_ = false; }

private:
    struct State {
        uint8_t* page;
        uint64_t used;
        bool failed;
    };
    static State& state() { static State s = {nullptr, 0, false}; return s; }
    static std::mutex& mutex() { static std::mutex m; return m; }
    int slot_ = 0;
    bool pending_ = false;
    hipStream_t stream_ = nullptr;
};
