// Host-only driver (tests/test_host_arrive.py): which decode calls sum their K
// splits inside the launch, with which arrival counters, and what the library
// does to its per-stream state.  The HIP calls that tl_api.cpp makes and the
// kernel launchers are stand-ins below: the "device" is host memory, a launch
// records what it was given, and a launch with counters leaves them as the
// kernel does.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "tl_internal.h"

static bool g_capturing = false;
static tl::DecodeLaunch g_last;
static int g_clears = 0;

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); std::memset(*p, 0xa5, n); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int*, hipDeviceAttribute_t, int) { return hipErrorInvalidValue; }
}

static float g_scratch[16];

namespace tl {
hipError_t launch_repack(const void*, void*, int64_t, int64_t, const Layout&, bool, hipStream_t) { std::abort(); }
hipError_t launch_decode(const DecodeLaunch& d, hipStream_t) {
    g_last = d;
    if (d.arrive)   // every split of every tile arrives; the other set is cleared
        for (int i = 0; i < kArriveTiles; ++i) d.arrive[d.arrive_clear + i * kArriveStride] = 0;
    return hipSuccess;
}
hipError_t launch_splitk_reduce(const DecodeLaunch&, hipError_t, hipStream_t) { std::abort(); }
hipError_t launch_lgms(const DecodeLaunch&, int64_t, int, hipStream_t) { std::abort(); }
int lgms_ctas_per_cu(int) { std::abort(); }
hipError_t launch_prefill(const PrefillLaunch&, hipStream_t) { return hipSuccess; }
hipError_t launch_view_load(const uint8_t*, int64_t, const ViewProgram&, uint8_t*, hipStream_t) { std::abort(); }
hipError_t launch_zero_u64(unsigned long long* p, hipStream_t) {
    ++g_clears;
    if (!g_capturing) std::memset(p, 0, kStateWords * sizeof *p);
    return hipSuccess;
}
hipError_t launch_stream_read(const uint8_t*, int64_t, unsigned*, hipStream_t) { std::abort(); }
hipError_t scratch_address(float** p) { *p = g_scratch; return hipSuccess; }
}  // namespace tl

using namespace tl;

static int bad = 0;
#define CHECK(x) do { if (!(x)) { ++bad; std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); } } while (0)

static const void* dp(int i) { return reinterpret_cast<const void*>(uintptr_t(i) << 42); }
static void* out() { return const_cast<void*>(dp(3)); }

// tl_gemm of these sizes on 'stream': the counters it was given
static unsigned* call(int kind, int elem, int64_t M, int64_t N, int64_t K, int S, int stream, bool noalloc = false, int fetch = 0) {
    tl_layout_desc d = {};
    d.kind = kind;
    d.elem_bytes = elem;
    d.G = 4096;
    d.block_rows = 32;
    d.split_k = S;
    g_last = DecodeLaunch();
    const int mode = (kind == TL_LAYOUT_TILE ? TL_FETCH_BLOCK : TL_FETCH_NATIVE) | fetch;
    void* s = reinterpret_cast<void*>(uintptr_t(stream));
    const int rc = noalloc ? tl_gemm_noalloc(dp(1), dp(2), out(), M, N, K, &d, mode, s)
                           : tl_gemm(dp(1), dp(2), out(), M, N, K, &d, mode, s);
    CHECK(rc == TL_OK);
    return g_last.arrive;
}

static bool zero(const unsigned* set) {
    for (int i = 0; i < kArriveTiles; ++i)
        if (set[i * kArriveStride]) return false;
    return true;
}

int main() {
    // the calls that are summed inside the launch: each layout and type, both
    // sides of every line
    CHECK(call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 1));
    CHECK(call(TL_LAYOUT_NK_ROW, 2, 1, 1024, 1024, 0, 1));
    CHECK(call(TL_LAYOUT_TILE, 1, 1, 1024, 2048, 0, 1));
    CHECK(call(TL_LAYOUT_NK_ROW, 1, 1, 1024, 2048, 0, 1));
    CHECK(call(TL_LAYOUT_KN_ROW, 2, 1, 1024, 4096, 2, 1));
    CHECK(call(TL_LAYOUT_TILE, 2, 16, 1024, 4096, 8, 1));       // 4096 floats per tile
    CHECK(!call(TL_LAYOUT_TILE, 2, 16, 1024, 4096, 9, 1));
    CHECK(!call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 1, 1));       // not split
    CHECK(!call(TL_LAYOUT_TILE, 2, 1, 4096, 4096, 4, 1));       // 32 MB
    CHECK(!call(TL_LAYOUT_TILE, 2, 8, 10240, 8192, 0, 1));
    CHECK(call(TL_LAYOUT_TILE, 2, 1, 4096, 1024, 2, 1));        // 256 workgroups, 128 tiles
    CHECK(!call(TL_LAYOUT_TILE, 2, 1, 4128, 1024, 2, 1));       // 258
    CHECK(!call(TL_LAYOUT_TILE, 2, 1, 8192, 1024, 3, 1));       // 768, of 4 waves
    CHECK(!call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 1, true)); // allocation-free: two launches

    // under capture those that are faster so on the GPU alone
    g_capturing = true;
    CHECK(call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 1));
    CHECK(!call(TL_LAYOUT_TILE, 1, 1, 1024, 2048, 0, 1));
    CHECK(!call(TL_LAYOUT_TILE, 2, 33, 1002, 1024, 2, 1));
    CHECK(call(TL_LAYOUT_TILE, 2, 33, 1004, 1024, 2, 1));
    CHECK(call(TL_LAYOUT_TILE, 2, 32, 1002, 1024, 2, 1));
    g_capturing = false;
    CHECK(call(TL_LAYOUT_TILE, 2, 33, 1002, 1024, 2, 1));

    // the two sets of counters are used in turn, on each stream its own, also
    // when other calls come between
    unsigned* a = call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 2);
    const int step = g_last.arrive_clear;
    call(TL_LAYOUT_TILE, 2, 8, 10240, 8192, 0, 2);
    unsigned* b = call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 2);
    CHECK(a && b && b == a + step && g_last.arrive_clear == -step);
    CHECK(call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 2) == a);
    CHECK(call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 1) != a);
    CHECK(zero(a) && zero(b));
    // a count left behind (a replay that overlapped a call) is gone two calls on
    b[5 * kArriveStride] = 1;
    a[7 * kArriveStride] = 3;
    call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 2);               // on b, clears a
    CHECK(zero(a));
    call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 2);               // on a, clears b
    CHECK(zero(b));

    // reading the tally clears the tally, and no counter
    unsigned long long* tally = reinterpret_cast<unsigned long long*>(step > 0 ? a : b) - kArriveAt;
    *tally = 42;
    a[9 * kArriveStride] = 1;
    int64_t bytes = 0;
    const int clears = g_clears;
    CHECK(tl_fetch_counter_read(reinterpret_cast<void*>(uintptr_t(2)), &bytes) == TL_OK && bytes == 42);
    CHECK(*tally == 0 && a[9 * kArriveStride] == 1 && g_clears == clears);

    // a state first made under capture: its clear is only recorded, so no call
    // relies on its counters
    g_capturing = true;
    CHECK(!call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 3));
    g_capturing = false;
    CHECK(!call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 3));
    tl_release();
    CHECK(call(TL_LAYOUT_TILE, 2, 1, 1024, 1024, 0, 3));
    tl_release();
    std::printf("host arrive driver: %d unexpected results\n", bad);
    return bad ? 1 : 0;
}
