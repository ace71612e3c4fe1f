// Device buffers of one visual-inertial call (host code).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

namespace gba {
namespace vi {

// Device buffers of one call, carved from a few allocations (an allocation
// and its release cost 20-200 us each; a solve takes about 50 buffers) and
// released on every return path.  Scratch buffers come from the far end of the
// same allocation (or one of their own) and are given back by drop_scratch();
// what takes their place is used on the same stream, after them.
struct DevBufs {
    std::vector<void*> chunks, scratch_own;
    char* at = nullptr;
    size_t left = 0, next, bytes = 0;
    size_t scratch_tail = 0;   // scratch bytes at the end of the current chunk
    explicit DevBufs(size_t expect) : next(expect) {}
    DevBufs(const DevBufs&) = delete;
    DevBufs& operator=(const DevBufs&) = delete;
    ~DevBufs() {
        drop_scratch();
        for (void* q : chunks) (void)hipFree(q);
    }
    void drop_scratch() {
        left += scratch_tail;
        scratch_tail = 0;
        for (void* q : scratch_own) (void)hipFree(q);
        scratch_own.clear();
    }
    template <typename T>
    bool scratch(T** dst, const T* src, size_t n) {
        const size_t need = (n * sizeof(T) + 16 + 255) & ~(size_t)255;
        if (need <= left) {
            left -= need;
            scratch_tail += need;
            *dst = (T*)(at + left);
        } else {
            void* q = nullptr;
            if (hipMalloc(&q, need) != hipSuccess) {
                (void)hipGetLastError();
                return false;
            }
            scratch_own.push_back(q);
            *dst = (T*)q;
        }
        return !src || n == 0 || hipMemcpy(*dst, src, n * sizeof(T), hipMemcpyHostToDevice) == hipSuccess;
    }
    template <typename T>
    bool up(T** dst, const T* src, size_t n) {
        const size_t need = (n * sizeof(T) + 16 + 255) & ~(size_t)255;
        if (need > left) {
            const size_t size = (std::max(need, next) + 255) & ~(size_t)255;   // (scratch starts from its end)
            void* q = nullptr;
            if (hipMalloc(&q, size) != hipSuccess) {
                // the expected size may be more than what is left needs
                const bool ok = size > need && hipMalloc(&q, need) == hipSuccess;
                (void)hipGetLastError();   // a failed allocation is the caller's to handle
                if (!ok) return false;
                left = need;
            } else {
                left = size;
            }
            chunks.push_back(q);
            bytes += left;
            at = (char*)q;
            scratch_tail = 0;   // (of a chunk that is not returned to)
            next = std::max<size_t>(next / 32, 1 << 20);
        }
        *dst = (T*)at;
        at += need;
        left -= need;
        return !src || n == 0 || hipMemcpy(*dst, src, n * sizeof(T), hipMemcpyHostToDevice) == hipSuccess;
    }
};

}  // namespace vi
}  // namespace gba
