// The host side of the trigger scans against a HIP runtime written here: the functions below take the place of the runtime's
// for libst.so, because the executable comes first in the order in which symbols are looked up.  No GPU is used; a "launch"
// evaluates the rule on the CPU from the kernel's arguments.  Exit status 0 if every check holds.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <vector>

#include "../../include/st.h"

static int g_device = 0;
static size_t g_lds = 0;  // dynamic LDS of the last launch
static int g_launches = 0, g_copies = 0;
// pinned memory: what the next allocation does, and the blocks held
enum Pinned { kWorks, kNoMemory, kNoAddress, kNullAddress };
static Pinned g_pinned = kWorks;
static int g_allocated = 0, g_held = 0;
static hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
static bool g_strict = false;  // an allocation or a release came under another capture mode than the relaxed one
alignas(256) static int32_t g_symbol[1 + ST_SCAN_STATIC_MAX_CAP];  // the library's static device array

extern "C" {
hipError_t hipGetDevice(int *d) { return *d = g_device, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t) {
    return ++g_copies, memcpy(dst, src, n), hipSuccess;
}

hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) { return std::swap(*m, g_mode), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    g_strict |= g_mode != hipStreamCaptureModeRelaxed;
    if (g_pinned == kNoMemory) return hipErrorOutOfMemory;
    return ++g_allocated, ++g_held, *p = malloc(n), hipSuccess;
}
hipError_t hipHostFree(void *p) {
    g_strict |= g_mode != hipStreamCaptureModeRelaxed;
    return --g_held, free(p), hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **dev, void *host, unsigned) {
    if (g_pinned == kNoAddress) return hipErrorInvalidValue;
    return *dev = g_pinned == kNullAddress ? nullptr : host, hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = g_symbol, hipSuccess; }

// What a launch would be: stored by the call that the compiler puts in front of a kernel's stub, read back by the stub.
static dim3 g_grid, g_block;
static size_t g_shared;
static hipStream_t g_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream) {
    return g_grid = grid, g_block = block, g_shared = shared, g_stream = stream, hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream) {
    return *grid = g_grid, *block = g_block, *shared = g_shared, *stream = g_stream, hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3 grid, dim3 block, void **args, size_t shared, hipStream_t) {
    if (grid.x != 1 || block.x != 1024) return hipErrorInvalidConfiguration;
    const auto *tokens = *(const int32_t **)args[0];
    const int lo = *(int *)args[1], hi = *(int *)args[2], window = *(int *)args[5], vocab = *(int *)args[6], cap = *(int *)args[8];
    const auto *kw = *(const uint32_t **)args[3], *delim = *(const uint32_t **)args[4];
    auto *positions = *(int32_t **)args[7], *n_found = *(int32_t **)args[9];
    auto in = [&](const uint32_t *bm, int id) { return id >= 0 && id < vocab && (bm[id >> 5] >> (id & 31) & 1u); };
    int n = 0;
    for (int p = lo; p < hi; ++p) {
        const int w = window - 1;
        bool fire = w == 0 && in(kw, tokens[p]);
        if (w > 0 && p >= w && in(delim, tokens[p - w])) {
            bool key = false, broken = false;
            for (int q = p - w + 1; q <= p; ++q) key |= in(kw, tokens[q]), broken |= q < p && in(delim, tokens[q]);
            fire = key && !broken;
        }
        if (fire && n < cap) positions[n] = p;
        n += fire;
    }
    *n_found = n;
    return ++g_launches, g_lds = shared, hipSuccess;
}
}  // extern "C"

#define CHECK(c)                                                                                             \
    do {                                                                                                     \
        if (!(c)) {                                                                                          \
            std::fprintf(stderr, "check failed at line %d: %s (%s)\n", __LINE__, #c, st_last_error());       \
            return 1;                                                                                        \
        }                                                                                                    \
    } while (0)

static std::vector<uint32_t> every(int step, int vocab) {
    std::vector<uint32_t> bm((vocab + 31) / 32);
    for (int i = 0; i < vocab; i += step) bm[i >> 5] |= 1u << (i & 31);
    return bm;
}

// A scan stages its bitmaps in LDS only where it walks more than one tile of 4096 positions and they fit.
static int short_scans_copy_no_bitmaps() {
    const int n = 40000;
    std::vector<int32_t> toks(n), out(n + 1);
    for (int i = 0; i < n; ++i) toks[i] = (int)((uint32_t)i * 2654435761u % 151936u);
    for (int vocab : {64, 151936, 600000})
        for (int window : {1, 2, 21}) {
            const auto kw = every(97, vocab), dl = every(89, vocab);
            const st_trigger_rule rule = {kw.data(), window > 1 ? dl.data() : nullptr, window, vocab};
            const size_t bytes = (size_t)((vocab + 31) / 32 + 3) / 4 * 16 * (window > 1 ? 2 : 1);
            for (int lo : {0, 5000})
                for (int len : {0, 1, 20, 300, 4075, 4096, 4097, 4608, 18000, 30000}) {
                    const int walked = len + (lo ? window - 1 : 0);
                    CHECK(st_trigger_scan(&rule, toks.data(), lo, lo + len, out.data() + 1, n, out.data(), nullptr, nullptr,
                                          ST_OUT_DEVICE) == ST_OK);
                    CHECK(g_lds == (walked > 4096 && bytes <= 61440 ? bytes : 0));
                }
        }
    return 0;
}

// st_trigger_scan_static on four GPUs, on three of which its pinned staging cannot be had: one block at most is held for each,
// later calls allocate nothing, and the device array in its place delivers the same, below and above what one copy brings back.
static int staging_with_and_without_pinned_memory() {
    const int n = 9000, vocab = 1000;
    std::vector<int32_t> toks(n);
    for (int i = 0; i < n; ++i) toks[i] = i * 7 % vocab;
    const auto kw = every(2, vocab);
    const st_trigger_rule rule = {kw.data(), nullptr, 1, vocab};
    for (Pinned how : {kWorks, kNoMemory, kNoAddress, kNullAddress}) {
        g_device = how, g_pinned = how, g_allocated = g_held = g_copies = 0;
        for (int hi : {9000, 300, 3000, 0})
            for (int cap : {4096, 1024, 5, 0}) {
                std::vector<int32_t> pos(cap + 1, -7);
                int32_t found = -1;
                CHECK(st_trigger_scan_static(&rule, toks.data(), 0, hi, pos.data(), cap, &found, nullptr) == ST_OK);
                int32_t k = 0;
                for (int p = 0; p < hi; ++p)
                    if (toks[p] % 2 == 0 && k++ < cap) CHECK(pos[k - 1] == p);
                CHECK(found == k && pos[k < cap ? k : cap] == -7);
                CHECK(g_allocated <= 1 && g_held == (how == kWorks) && (g_copies == 0) == (how == kWorks));
            }
        CHECK(!g_strict && g_mode == hipStreamCaptureModeGlobal);
    }
    return g_device = 0;
}

int main() {
    if (short_scans_copy_no_bitmaps() || staging_with_and_without_pinned_memory()) return 1;
    std::printf("ok\n");
    return 0;
}
