// slab.h -- many arrays out of one device allocation.  An allocation of a
// megabyte or more and its release take some 55 us together, a small one 3 us:
// forty of them were a quarter of preparing a 2,000-vertex graph and 3 ms of
// preparing 50,000 vertices.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ebb {

inline size_t slab_round(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

// Bytes of a slab holding arrays taken one after the other.
struct SlabSize {
    size_t bytes = 0;
    template <typename T>
    SlabSize& add(int64_t n, int copies = 1) {
        bytes += copies * slab_round(sizeof(T) * (size_t)(n > 0 ? n : 1));
        return *this;
    }
};

// Owns its memory until release().
struct Slab {
    char* base = nullptr;
    size_t used = 0, cap = 0;
    Slab() = default;
    Slab(const Slab&) = delete;
    Slab& operator=(const Slab&) = delete;
    ~Slab() { if (base) (void)hipFree(base); }
    hipError_t init(const SlabSize& s) {
        const hipError_t e = hipMalloc((void**)&base, s.bytes ? s.bytes : 256);
        if (e != hipSuccess) base = nullptr;
        cap = base ? s.bytes : 0;
        return e;
    }
    char* release() { char* p = base; base = nullptr; return p; }
};

// An array of a slab.
template <typename T>
struct SBuf {
    T* p = nullptr;
    hipError_t alloc(Slab& s, int64_t n) {
        const size_t bytes = slab_round(sizeof(T) * (size_t)(n > 0 ? n : 1));
        if (s.used + bytes > s.cap) return hipErrorOutOfMemory;
        p = reinterpret_cast<T*>(s.base + s.used);
        s.used += bytes;
        return hipSuccess;
    }
};

}  // namespace ebb
