// Host-only helper, free of HIP so that it can be tested by itself.
#pragma once
#include <cstddef>
#include <mutex>
#include <vector>

namespace gcn {

// Buffers for partial results, those of a device and stream apart from all others.  A call takes one and gives it back once it has queued its work:
// what the next call with that buffer queues runs behind it, on the same stream.  Calls from several threads on one stream have a buffer each
// while they overlap, since their launches may alternate; so there are as many as calls have overlapped.  A buffer that is too small is replaced, and
// kept until clear(): work that was queued or captured earlier may use it.
class ScratchPool {
public:
    // alloc(&p, bytes) returns 0 or an error, which is handed on
    template <class Alloc>
    int take(int device, const void* stream, size_t bytes, void** p, const Alloc& alloc) {
        std::lock_guard<std::mutex> lk(mu_);
        Buffer* best = nullptr;                     // the smallest that will do, else the largest
        for (Buffer& b : buffers_) {
            if (b.out || b.device != device || b.stream != stream) continue;
            const bool does = b.bytes >= bytes;
            if (!best || (does ? best->bytes < bytes || b.bytes < best->bytes : best->bytes < bytes && b.bytes > best->bytes)) best = &b;
        }
        if (!best || best->bytes < bytes) {
            void* fresh = nullptr;
            const size_t want = bytes + bytes / 4;
            if (const int rc = alloc(&fresh, want)) return rc;
            if (!best) {
                buffers_.push_back({device, stream, nullptr, 0, false});
                best = &buffers_.back();
            } else {
                retired_.push_back(best->p);
            }
            best->p = fresh;
            best->bytes = want;
        }
        best->out = true;
        *p = best->p;
        return 0;
    }
    void give(const void* p) {
        std::lock_guard<std::mutex> lk(mu_);
        for (Buffer& b : buffers_)
            if (b.p == p) b.out = false;
    }
    template <class Free>
    void clear(const Free& free) {
        std::lock_guard<std::mutex> lk(mu_);
        for (const Buffer& b : buffers_) free(b.p);
        for (void* p : retired_) free(p);
        buffers_.clear();
        retired_.clear();
    }

private:
    struct Buffer {
        int device;
        const void* stream;
        void* p;
        size_t bytes;
        bool out;
    };
    std::mutex mu_;
    std::vector<Buffer> buffers_;
    std::vector<void*> retired_;
};

}  // namespace gcn
