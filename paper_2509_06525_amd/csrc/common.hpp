// Internal helpers shared by the library's translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <deque>
#include <string>

#include "tbkpm.h"

namespace tbk {

// Thread-local error text behind tbk_last_error().
void set_error(const char *fmt, ...);
void clear_error();

// Returns the status and records the message.
tbk_status fail(tbk_status st, const char *fmt, ...);

#define TBK_HIP(call)                                                                 \
    do {                                                                              \
        hipError_t e_ = (call);                                                       \
        if (e_ != hipSuccess)                                                         \
            return ::tbk::fail(TBK_ERR_DEVICE, "%s failed: %s (%s:%d)", #call,        \
                               hipGetErrorString(e_), __FILE__, __LINE__);            \
    } while (0)

#define TBK_CHECK(cond, st, ...)                                                      \
    do {                                                                              \
        if (!(cond)) return ::tbk::fail((st), __VA_ARGS__);                           \
    } while (0)

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

class Arena;

// Stream-ordered temporary device buffer, freed on scope exit (or with its arena).
class DevBuf {
  public:
    DevBuf() = default;
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    ~DevBuf() { release(); }
    hipError_t alloc(size_t bytes, hipStream_t s) {
        release();
        stream_ = s;
        bytes_ = bytes ? bytes : 256;
        return hipMallocAsync(&p_, bytes_, s);
    }
    hipError_t alloc(size_t bytes, Arena &arena);
    void release() {
        if (p_ && !borrowed_) (void)hipFreeAsync(p_, stream_);
        p_ = nullptr;
        borrowed_ = false;
    }
    template <class T> T *as() const { return static_cast<T *>(p_); }
    size_t bytes() const { return bytes_; }

  private:
    void *p_ = nullptr;
    size_t bytes_ = 0;
    hipStream_t stream_ = nullptr;
    bool borrowed_ = false;
};

// Temporary buffers of one call, carved from blocks that are freed with it.  A
// hipFreeAsync takes the host 10-20 us whatever its size, and a few hundred where the
// pool maps or unmaps memory (a learned build of 590,000 atoms made 44 of them, 3 ms
// of its 4.4): the first block is meant to hold all of a call's buffers.
class Arena {
  public:
    Arena() = default;
    Arena(const Arena &) = delete;
    Arena &operator=(const Arena &) = delete;
    // The call takes about `bytes` on stream s: the size of the first block.
    void expect(size_t bytes, hipStream_t s) {
        next_ = bytes;
        stream_ = s;
    }
    hipError_t take(size_t bytes, void **p) {
        bytes = (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
        if (blocks_.empty() || used_ + bytes > blocks_.back().bytes()) {
            const hipError_t e = grow(bytes);
            if (e != hipSuccess) return e;
        }
        *p = blocks_.back().as<char>() + used_;
        used_ += bytes;
        return hipSuccess;
    }
    hipStream_t stream() const { return stream_; }

  private:
    hipError_t grow(size_t bytes) {
        used_ = 0;
        blocks_.emplace_back();
        const hipError_t e = blocks_.back().alloc(std::max(bytes, next_), stream_);
        next_ = (size_t)1 << 20;
        if (e != hipSuccess) blocks_.pop_back();
        return e;
    }
    std::deque<DevBuf> blocks_;
    size_t used_ = 0, next_ = 0;
    hipStream_t stream_ = nullptr;
};

inline hipError_t DevBuf::alloc(size_t bytes, Arena &arena) {
    release();
    const hipError_t e = arena.take(bytes, &p_);
    if (e != hipSuccess) return e;
    borrowed_ = true;
    stream_ = arena.stream();
    bytes_ = bytes;
    return hipSuccess;
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Number of XCDs of an MI355X; workgroups are dispatched round-robin over them.
constexpr int kNumXcd = 8;

}  // namespace tbk
