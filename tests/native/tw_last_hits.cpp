// The window loop's hit ranges where the call's hits end at `end`, up to 2^31 - 1:
// next_window and collect, by one wave, against a serial scan. The arrays are
// address space only (a page is backed once it is touched), with as much that
// cannot be read in front of them, so that an index that wraps ends the program.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <sys/mman.h>
#include <thread>
#include <vector>

#include "hough_tw.h"

using namespace hough;

template <class T>
T *array(int64_t n) {
    const size_t bytes = ((size_t)n + 4096) * sizeof(T);
    char *p = (char *)mmap(nullptr, 2 * bytes, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    const size_t half = (bytes + 4095) & ~(size_t)4095;
    if (p == MAP_FAILED || mprotect(p + half, 2 * bytes - half, PROT_READ | PROT_WRITE) != 0) {
        std::perror("mmap");
        std::exit(2);
    }
    return (T *)(p + half);
}

int main(int argc, char **argv) {
    const int64_t end = std::atoll(argv[1]);
    const int n = std::atoi(argv[2]);   // hits of the last timeline
    const int64_t base = end - n;
    TwArgs A{};
    float *t = array<float>(end), *z = array<float>(end);
    int16_t *vane = array<int16_t>(end);
    A.t = t;
    A.z = z;
    A.vane = vane;
    A.used = array<int32_t>(end);
    A.wz = array<float>(end);
    A.wv = array<int16_t>(end);
    A.widx = array<int32_t>(end);
    A.window_ns = 10.0f;
    A.step_ns = 5.0f;
    A.n_windows = 60;
    for (int i = 0; i < n; ++i) {   // busy at first and last, empty between
        t[base + i] = i < n / 2 ? 0.25f * i : 200.0f + 0.01f * i;
        z[base + i] = (float)i;
        A.used[base + i] = i % 5 == 0 ? 1 : -1;
    }
    struct Seen {
        int w, wa, we, n;
    };
    std::vector<Seen> got;
    tw::Shared T{};
    T.wa = (int)base;
    std::vector<std::thread> wave;
    for (unsigned l = 0; l < 64; ++l)
        wave.emplace_back([&, l] {
            threadIdx = {l, 0, 0};
            for (;;) {
                tw::next_window(A, 3u, T, (int)end);
                __syncthreads();
                if (!T.busy) break;
                const int c = tw::collect<64>(A, T, T.wa, T.we, base);
                __syncthreads();
                if (l == 0) {
                    got.push_back({T.w, T.wa, T.we, c});
                    ++T.w;
                }
                __syncthreads();
            }
        });
    for (auto &x : wave) x.join();
    // every window with at least three unused hits was seen, with its range and hits
    size_t k = 0;
    for (int w = 0; w < A.n_windows; ++w) {
        const float lo = (float)w * A.step_ns, hi = lo + A.window_ns;
        int64_t a = base, e = base;
        while (a < end && t[a] < lo) ++a;
        while (e < end && t[e] < hi) ++e;
        int unused = 0;
        for (int64_t i = a; i < e; ++i) unused += A.used[i] < 0;
        while (k < got.size() && got[k].w < w) ++k;
        const bool seen = k < got.size() && got[k].w == w;
        if (unused >= 3 && !seen) return std::printf("window %d missed\n", w), 1;
        if (seen && (got[k].wa != a || got[k].we != e || got[k].n != unused))
            return std::printf("window %d: [%d, %d) %d, not [%lld, %lld) %d\n", w, got[k].wa, got[k].we, got[k].n,
                               (long long)a, (long long)e, unused), 1;
    }
    if (got.empty()) return std::printf("no window\n"), 1;
    std::printf("ok %zu windows\n", got.size());
    return 0;
}
