// Device buffers of a context and how they follow a mesh's size.  The caller
// declares hipMalloc, hipFree, hipMemcpy and hipGetLastError (the HIP runtime;
// a CPU test gives its own).
#pragma once

#include <algorithm>
#include <cstddef>
#include <utility>

namespace dgx {

template <typename T>
struct DevBuf {
    T *p = nullptr;
    size_t n = 0;    // elements in use
    size_t cap = 0;  // elements allocated
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        n = cap = 0;
    }
};

template <typename T>
bool buf_alloc(DevBuf<T> &b, size_t n, size_t cap) {
    void *p = nullptr;
    if (hipMalloc(&p, cap * sizeof(T)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    b.p = (T *)p;
    b.n = n;
    b.cap = cap;
    return true;
}

// Exactly n elements; false (and an empty buffer) where memory is short.
template <typename T>
bool buf_exact(DevBuf<T> &b, size_t n) {
    if (b.p && b.n == n && b.cap == n) return true;
    b.release();
    return n == 0 || buf_alloc(b, n, n);
}

// The same for the buffers that follow the mesh's size, whose users a mesh
// change waits for: one that is large enough stays while it is at most
// kMeshSlack larger than needed, and one that has to grow takes an eighth
// more, up to kMeshSlack, where there is memory for it.  (An adaptation cycle
// changes some twenty of them by a few percent; a free and an allocation take
// 60 us and more.)  The slack is never what a call fails for: a caller that is
// refused here gives all of it back (release, or buf_trim for the buffers still
// in use) and asks again.
constexpr size_t kMeshSlack = (size_t)32 << 20;
template <typename T>
bool buf_keeps(const DevBuf<T> &b, size_t n) {
    return b.p && n > 0 && b.cap >= n && b.cap - n <= kMeshSlack / sizeof(T);
}
template <typename T>
bool buf_mesh(DevBuf<T> &b, size_t n) {
    const size_t slack = kMeshSlack / sizeof(T);
    if (buf_keeps(b, n)) {
        b.n = n;
        return true;
    }
    const bool grows = b.p && n > b.cap;
    b.release();
    if (grows && buf_alloc(b, n, n + std::min(n / 8, slack))) return true;
    return buf_exact(b, n);
}

// Gives a buffer's slack back, its contents kept (the device has been waited
// for), where a copy of them fits.
template <typename T>
void buf_trim(DevBuf<T> &b) {
    DevBuf<T> c;
    if (!b.p || b.cap == b.n || !buf_alloc(c, b.n, b.n)) return;
    if (hipMemcpy(c.p, b.p, b.n * sizeof(T), hipMemcpyDeviceToDevice) != hipSuccess) {
        (void)hipGetLastError();
        c.release();
        return;
    }
    std::swap(b, c);
    c.release();
}

}  // namespace dgx
