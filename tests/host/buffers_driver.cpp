// CPU driver of the device buffers (csrc/host_buffers.h) for the tests, over a
// card of a given number of bytes.  Reads the card's size, then commands over
// eight buffers of doubles:
//
//   mesh i n    buf_mesh      exact i n   buf_exact
//   trim i      buf_trim      free i      release
//
// and prints for each: whether it succeeded, the elements in use and allocated,
// the bytes in use on the card, and whether the first and last element in use
// are what the driver wrote there when it last asked for the buffer.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <map>
#include <string>

enum hipError_t { hipSuccess, hipErrorOutOfMemory };
enum hipMemcpyKind { hipMemcpyDeviceToDevice };
static size_t card, used;
static std::map<void *, size_t> live;
static hipError_t hipMalloc(void **p, size_t n) {
    if (used + n > card) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    live[*p] = n;
    used += n;
    return hipSuccess;
}
static hipError_t hipFree(void *p) {
    used -= live.at(p);
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
static hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    if (n > live.at(d)) std::abort();
    std::memcpy(d, s, n);
    return hipSuccess;
}
static hipError_t hipGetLastError() { return hipSuccess; }

#include "../../paper_2511_17551_amd/csrc/host_buffers.h"

int main() {
    dgx::DevBuf<double> buf[8];
    double mark[8] = {};
    std::cin >> card;
    std::string cmd;
    int i, turn = 0;
    while (std::cin >> cmd >> i) {
        dgx::DevBuf<double> &b = buf[i];
        bool ok = true;
        if (cmd == "mesh" || cmd == "exact") {
            size_t n;
            std::cin >> n;
            ok = cmd == "mesh" ? dgx::buf_mesh(b, n) : dgx::buf_exact(b, n);
            mark[i] = ++turn;
            if (b.p) b.p[0] = b.p[b.n - 1] = mark[i];
        } else if (cmd == "trim") {
            dgx::buf_trim(b);
        } else {
            b.release();
        }
        const bool kept = !b.p || (b.p[0] == mark[i] && b.p[b.n - 1] == mark[i]);
        std::printf("%d %zu %zu %zu %d\n", ok, b.n, b.cap, used, kept);
    }
    for (auto &b : buf) b.release();
    return used != 0;
}
