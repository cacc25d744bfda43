// Token-level takeover trigger (paper Section 3 (1), keyword sets of Appendix C as id bitmaps; window > 2
// is the n1-token sentence after a delimiter): an ordered, exact scan of a token range.
//
// The rule is evaluated as two running maxima instead of a look-back loop per position.  With w = window - 1,
//   lastD(q) = largest index j <= q whose token is a delimiter (-1: none),
//   lastK(q) = largest index j <= q whose token is a keyword   (-1: none),
// position p fires exactly when  p - w >= 0,  lastD(p - 1) == p - w  (a delimiter right before the sentence and none
// inside it before its last token)  and  lastK(p) > p - w  (a keyword inside it).  Both maxima are prefix scans, so
// a position costs O(1) whatever the window; the scan starts w tokens before `lo`, which is as far back as any
// position of the range looks.  One 1024-thread block walks the tokens in tiles, carries the two maxima from tile
// to tile and compacts the firing positions in ascending order with wave ballots.
#include <cstring>
#include <mutex>

#include "st_device.h"
#include "st_internal.h"

namespace st {

__device__ __forceinline__ bool in_set(const uint32_t *bm, int id, int vocab) {
    return id >= 0 && id < vocab && ((bm[id >> 5] >> (id & 31)) & 1u);
}

// inclusive running maximum over the lanes of a wave: shifts inside the rows of 16 lanes, then the last lane of a row to the
// rows after it (a lane without a source keeps its value)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_max(int v) {
    return max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ int wave_running_max(int v) {
    v = dpp_max<0x111, 0xf>(v);  // row_shr:1
    v = dpp_max<0x112, 0xf>(v);  // row_shr:2
    v = dpp_max<0x114, 0xf>(v);  // row_shr:4
    v = dpp_max<0x118, 0xf>(v);  // row_shr:8
    v = dpp_max<0x142, 0xa>(v);  // row_bcast15 into rows 1 and 3
    return dpp_max<0x143, 0xc>(v);  // row_bcast31 into rows 2 and 3
}

// A thread owns PER consecutive positions of a tile of 1024 * PER: one block's chain of tiles is bound by the latency of a
// tile (token load, bitmap look-ups, two barriers) and by the look-ups, random 4-byte reads that a CU serves one lane a clock.
// STAGED: both bitmaps are copied to LDS first, beside the token load (a vocabulary of 152 k ids takes 19 KB each), and looked
// up there.  scan_form says which scan takes which form, and why.
constexpr size_t kScanLds = 60 << 10;  // with the kernel's own arrays below the 64 KB every kernel may use

template <int PER, bool STAGED>
__global__ __launch_bounds__(1024) void k_trigger_scan(const int32_t *__restrict__ tokens, int lo, int hi,
                                                       const uint32_t *kw, const uint32_t *delim, int window, int vocab,
                                                       int32_t *__restrict__ positions, int cap,
                                                       int32_t *__restrict__ n_found) {
    constexpr int kTile = 1024 * PER, kBits = PER == 8 ? 4 : 3;  // bits of a count of 0 .. PER
    static_assert(PER == 4 || PER == 8, "bits of a thread's count");
    __shared__ int wave_d[16], wave_k[16], wave_n[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int w = window - 1;
    const int scan_from = w == 0 ? lo : max(0, lo - w);
    int carry_d = -1, carry_k = -1, base = 0;  // the same in every thread
    auto fetch = [&](int start, int (&id)[PER]) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const uint32_t p = (uint32_t)start + threadIdx.x * PER + e;  // (a tile may end past 2^31)
            id[e] = p < (uint32_t)hi ? tokens[p] : -1;  // -1 belongs to no set
        }
    };
    int id[PER];
    if (scan_from < hi) fetch(scan_from, id);
    extern __shared__ __align__(16) uint32_t bitmaps[];
    if constexpr (STAGED) {
        const int words = (vocab + 31) >> 5, pad = (words + 3) & ~3;
        auto stage = [&](const uint32_t *src, uint32_t *dst) {
            const int n4 = ((uintptr_t)src & 15) == 0 ? words >> 2 : 0;
            for (int i = threadIdx.x; i < n4; i += 1024)
                reinterpret_cast<u32x4 *>(dst)[i] = reinterpret_cast<const u32x4 *>(src)[i];
            for (int i = 4 * n4 + threadIdx.x; i < words; i += 1024) dst[i] = src[i];
        };
        stage(kw, bitmaps);
        kw = bitmaps;
        if (w > 0) {
            stage(delim, bitmaps + pad);
            delim = bitmaps + pad;
        }
        __syncthreads();
    }
    for (long start = scan_from; start < hi; start += kTile) {
        const uint32_t p0 = (uint32_t)start + threadIdx.x * PER;  // positions past `hi` hold no token and never fire
        bool is_k[PER], is_d[PER];
        int own_d = -1, own_k = -1;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            is_k[e] = in_set(kw, id[e], vocab), is_d[e] = w > 0 && in_set(delim, id[e], vocab);
            if (is_d[e]) own_d = (int)(p0 + e);
            if (is_k[e]) own_k = (int)(p0 + e);
        }
        if (start + kTile < hi) fetch((int)start + kTile, id);  // under this tile's reductions
        const int run_d = wave_running_max(own_d), run_k = wave_running_max(own_k);
        int last_d = __shfl_up(run_d, 1, kWave), last_k = __shfl_up(run_k, 1, kWave);  // of the lanes before this one
        if (lane == 0) last_d = last_k = -1;
        if (lane == kWave - 1) wave_d[wave] = run_d, wave_k[wave] = run_k;
        __syncthreads();
        int all_d = carry_d, all_k = carry_k;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if (v == wave) last_d = max(last_d, all_d), last_k = max(last_k, all_k);  // everything before this wave
            all_d = max(all_d, wave_d[v]), all_k = max(all_k, wave_k[v]);
        }
        carry_d = all_d, carry_k = all_k;
        unsigned fire = 0;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int p = (int)(p0 + e);  // below `lo` if it has wrapped
            if (is_k[e]) last_k = p;
            // here last_d is the last delimiter before p, last_k the last keyword up to p
            const bool f = p >= lo && p < hi && (w == 0 ? is_k[e] : (p - w >= 0 && last_d == p - w && last_k > p - w));
            fire |= (unsigned)f << e;
            if (is_d[e]) last_d = p;
        }
        const int cnt = __popc(fire);  // its bits are summed over the lower lanes by ballots
        const unsigned long long below = (1ull << lane) - 1ull;
        int off = 0, wave_total = 0;
#pragma unroll
        for (int b = 0; b < kBits; ++b) {
            const unsigned long long m = __ballot(cnt >> b & 1);
            off += __popcll(m & below) << b, wave_total += __popcll(m) << b;
        }
        if (lane == 0) wave_n[wave] = wave_total;
        __syncthreads();
        int all_n = base;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if (v == wave) off += all_n;
            all_n += wave_n[v];
        }
        base = all_n;
#pragma unroll
        for (int e = 0; e < PER; ++e)
            if (fire >> e & 1u) {
                if (off < cap) positions[off] = (int)(p0 + e);
                ++off;
            }
        // (wave_d and wave_k were read before the second barrier, and wave_n is next written behind the next tile's first)
    }
    if (threadIdx.x == 0) *n_found = base;
}

// Copies the result (count and positions, contiguous on the device: count first) to the host: one copy and one wait for
// up to kScanFirst positions, the rest in a second one.  (Count and positions in turn cost a second round trip: 57 against
// 34 us for a scan of 4608 tokens with its call.)
constexpr int kScanFirst = 1024;
int deliver_scan(const int32_t *dev, int32_t range, int32_t *positions, int32_t cap, int32_t *n_found, hipStream_t s) {
    int32_t host[1 + kScanFirst];
    int32_t most = cap < range ? cap : range;
    const int32_t first = most < kScanFirst ? most : kScanFirst;
    hipError_t e = hipMemcpyAsync(host, dev, sizeof(int32_t) * (1 + (size_t)first), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ST_EHIP, "reading the scan's result back: %s", hipGetErrorString(e));
    *n_found = host[0];
    const int32_t k = host[0] < cap ? host[0] : cap, now = k < first ? k : first;
    if (now > 0) memcpy(positions, host + 1, sizeof(int32_t) * (size_t)now);
    if (k > now) {
        e = hipMemcpyAsync(positions + now, dev + 1 + now, sizeof(int32_t) * (size_t)(k - now), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return fail(ST_EHIP, "reading the positions back: %s", hipGetErrorString(e));
    }
    return ST_OK;
}

// The form of a scan that walks n positions with bitmaps of `lds` bytes.  Kernel alone, us, delimiter rule at 152 k ids (38 KB):
//   positions           1000   4000   4097   5000   6000   8000   9000  12289  14000  18000  24000  30000
//   4, not staged        4.5    6.0    8.1    8.7    8.9   10.1   13.0   16.9   17.8   22.2   27.8   35.5
//   8, not staged        6.0    7.4    7.4    8.2    9.1   11.1   15.9   17.6   19.2   25.6   29.3   36.7
//   4, staged            4.5    5.5    7.7    7.7    7.8    8.2   10.5   13.2   13.3   16.2   19.4   24.6
//   8, staged            5.5    6.9    7.0    7.5    8.0    9.0   12.3   12.9   13.2   17.7   19.6   23.8
// (4.2 is the rate of launches.)  So: one tile of four positions a thread unstaged, as short a kernel as there is; longer scans
// four and staged; eight where they save the last tile of four and that one is short (unstaged only the second tile is worth
// their slower look-ups), and in chains so long that whole tiles count.
struct ScanForm {
    int per;
    bool staged;
};
static ScanForm scan_form(long n, size_t lds) {
    const bool staged = n > 4096 && lds <= kScanLds;
    const long last = (n - 1) % 8192 + 1;  // positions of the last tile at eight a thread
    const bool saves = last > 4096 && last <= (n > 8192 ? 6144 : 5632);
    const bool wide = staged ? saves || n > 24576 : saves && n <= 8192;
    return {wide ? 8 : 4, staged};
}

void launch_trigger_scan(const st_trigger_rule &rule, const int32_t *tokens, int32_t lo, int32_t hi,
                         int32_t *positions, int32_t cap, int32_t *n_found, hipStream_t stream) {
    const int w = rule.window - 1;
    const size_t lds = (size_t)(((rule.vocab + 31ll) / 32 + 3) & ~3ll) * sizeof(uint32_t) * (w > 0 ? 2 : 1);
    const ScanForm f = scan_form((long)hi - (lo > w ? lo - w : 0), lds);
#define ST_SCAN(PERV, STAGEDV)                                                                                             \
    hipLaunchKernelGGL((k_trigger_scan<PERV, STAGEDV>), dim3(1), dim3(1024), STAGEDV ? lds : 0, stream, tokens, lo, hi,    \
                       rule.kw_bitmap, rule.delim_bitmap, rule.window, rule.vocab, positions, cap, n_found)
    if (f.per == 8 && f.staged) ST_SCAN(8, true);
    else if (f.per == 8) ST_SCAN(8, false);
    else if (f.staged) ST_SCAN(4, true);
    else ST_SCAN(4, false);
#undef ST_SCAN
}

// ---------------------------------------------------------------------------------------
// The scan for callers that cannot allocate device memory: the result staging (count + positions) belongs to the library --
// pinned host memory the kernel writes straight into, so that no copy follows it (4608 tokens with their call: 33.5 us with a
// device array and a copy, 22.8 us this way; 18000 tokens 49 and 35 us).  One per GPU the library has been called on, allocated
// by the first call, held until the process ends.  Where it cannot be had, a file-scope device array and a copy take its place.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) int32_t scratch[1 + ST_SCAN_STATIC_MAX_CAP];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
struct ScanStage {
    int32_t *dev, *host;  // where the kernel writes; the same memory as the host reads it (nullptr: device array)
};
static ScanStage g_stage[kMaxDevices];  // dev == nullptr: not looked up yet

static int scan_stage(ScanStage *out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(ST_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(ST_EHIP, "device index %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    ScanStage &st = g_stage[dev];
    if (!st.dev) {
        // (an allocation must not disturb a capture this thread may have under way on some stream)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool exchanged = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        void *host = nullptr, *p = nullptr;
        e = hipHostMalloc(&host, sizeof(scratch), hipHostMallocDefault);
        if (e == hipSuccess) {
            e = hipHostGetDevicePointer(&p, host, 0);
            if (e != hipSuccess || !p) (void)hipHostFree(host), p = nullptr;
        }
        if (exchanged) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e == hipSuccess && p) {
            st.dev = static_cast<int32_t *>(p), st.host = static_cast<int32_t *>(host);
        } else {
            (void)hipGetLastError();
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p)
                return fail(ST_EHIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
            st.dev = static_cast<int32_t *>(p), st.host = nullptr;
        }
    }
    *out = st;
    return ST_OK;
}

}  // namespace st

using namespace st;

extern "C" int st_trigger_scan_static(const st_trigger_rule *rule, const int32_t *tokens, int32_t lo, int32_t hi,
                                      int32_t *positions, int32_t cap, int32_t *n_found, void *stream) {
    if (!rule || !rule->kw_bitmap || !tokens || !n_found) return fail(ST_EINVAL, "rule, bitmap, tokens or n_found is NULL");
    if (rule->window < 1 || rule->window > ST_MAX_SCAN_WINDOW)
        return fail(ST_EINVAL, "window must be in [1, %d]", ST_MAX_SCAN_WINDOW);
    if (rule->window >= 2 && !rule->delim_bitmap) return fail(ST_EINVAL, "a window above 1 needs a delimiter bitmap");
    if (rule->vocab <= 0) return fail(ST_EINVAL, "rule vocab must be positive");
    if (cap < 0 || (cap > 0 && !positions)) return fail(ST_EINVAL, "cap < 0, or positions is NULL with cap > 0");
    if (cap > ST_SCAN_STATIC_MAX_CAP)
        return fail(ST_ERANGE, "cap %d exceeds the staging (%d positions)", cap, ST_SCAN_STATIC_MAX_CAP);
    if (lo < 0 || hi < lo) return fail(ST_ERANGE, "bad range [%d,%d)", lo, hi);
    ScanStage stage;
    if (int rc = scan_stage(&stage)) return rc;
    hipStream_t s = (hipStream_t)stream;
    // the kernel writes the count and the first min(count, cap) positions on every call: nothing of the previous
    // call's contents is read, so nothing has to be cleared
    launch_trigger_scan(*rule, tokens, lo, hi, stage.dev + 1, cap, stage.dev, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ST_EHIP, "trigger scan: %s", hipGetErrorString(e));
    if (!stage.host) return deliver_scan(stage.dev, hi - lo, positions, cap, n_found, s);
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ST_EHIP, "trigger scan: %s", hipGetErrorString(e));
    *n_found = stage.host[0];
    const int32_t k = stage.host[0] < cap ? stage.host[0] : cap;
    if (k > 0) memcpy(positions, stage.host + 1, sizeof(int32_t) * (size_t)k);
    return ST_OK;
}
