// Test program: launches that the runtime refuses (hipLaunchKernel is replaced here; a refused one never reaches it) must
// leave the device's count of waves in flight as they found it, or every later launch would be kept
// to one lane per chain.  Each call is made with its first, second, ... launch refused until one more than it has; after each
// the count is 0 and the same call, undisturbed, gives the same bytes.
// Linked against the library; prints a line per call and "refused launches: OK".
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <vector>

#include "../../include/lorenz_cipher.h"

static long g_refuse = -1;    // launches to let through before one is refused; -1: none is
static bool g_refused = false, g_pending = false;

extern "C" hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 wg, void **args, size_t lds, hipStream_t s) {
    static auto real = (hipError_t(*)(const void *, dim3, dim3, void **, size_t, hipStream_t))dlsym(RTLD_NEXT, "hipLaunchKernel");
    if (g_refuse == 0) {
        g_refuse = -1;
        g_refused = g_pending = true;
        return hipErrorLaunchOutOfResources;
    }
    if (g_refuse > 0) --g_refuse;
    return real(f, grid, wg, args, lds, s);
}

extern "C" hipError_t hipGetLastError(void) {
    static auto real = (hipError_t(*)())dlsym(RTLD_NEXT, "hipGetLastError");
    if (g_pending) {
        g_pending = false;
        return hipErrorLaunchOutOfResources;
    }
    return real();
}

#define NEED(x)                                                                                            \
    do {                                                                                                   \
        if (!(x)) {                                                                                        \
            std::printf("line %d: %s (%s)\n", __LINE__, #x, lz_last_error());                              \
            std::exit(1);                                                                                  \
        }                                                                                                  \
    } while (0)

static lz_ctx *ctx;
static uint8_t *in, *out;

static std::vector<uint8_t> bytes(size_t n) {
    std::vector<uint8_t> h(n);
    NEED(hipDeviceSynchronize() == hipSuccess);
    NEED(hipMemcpy(h.data(), out, n, hipMemcpyDeviceToHost) == hipSuccess);
    return h;
}

static uint32_t waves() {
    uint32_t w = 0;
    NEED(hipDeviceSynchronize() == hipSuccess);
    NEED(lz_unit_waves(ctx, &w, nullptr) == LZ_OK);
    return w;
}

static void check(const char *name, size_t n, const std::function<int()> &call) {
    NEED(call() == LZ_OK);
    const auto want = bytes(n);
    NEED(waves() == 0);
    int k = 0;
    for (;; ++k) {
        g_refuse = k;
        g_refused = false;
        const int rc = call();
        g_refuse = -1;
        g_pending = false;
        if (!g_refused) {
            NEED(rc == LZ_OK);
            break;
        }
        NEED(rc == LZ_E_HIP);
        const uint32_t w = waves();
        if (w != 0) {
            std::printf("%s: launch %d refused: %d waves stay counted\n", name, k, (int)w);
            std::exit(1);
        }
        NEED(call() == LZ_OK);
        NEED(bytes(n) == want);
    }
    std::printf("%s: %d launches\n", name, k);
    std::fflush(stdout);
}

int main() {
    constexpr size_t MAX = 20000000;
    const uint8_t pw[] = "refused";
    lz_params prm;
    NEED(lz_params_default(&prm) == LZ_OK);
    prm.n_it = 500;  // enough that rounds pay
    NEED(lz_context_create(0, &prm, &ctx) == LZ_OK);
    NEED(hipMalloc(&in, MAX) == hipSuccess && hipMalloc(&out, MAX + LZ_TAG_BYTES) == hipSuccess);
    std::vector<uint8_t> h(MAX);
    for (size_t i = 0; i < MAX; ++i) h[i] = (uint8_t)(i * 2654435761u >> 13);
    NEED(hipMemcpy(in, h.data(), MAX, hipMemcpyHostToDevice) == hipSuccess);
    for (size_t n : {(size_t)100, (size_t)65536, (size_t)3000000, (size_t)6000000, (size_t)1300000, MAX}) {
        char name[64];
        std::snprintf(name, sizeof name, "message of %zu", n);
        check(name, n + LZ_TAG_BYTES, [&] { return lz_encrypt(ctx, pw, 7, in, n, out, nullptr); });
        std::snprintf(name, sizeof name, "stream of %zu", n);
        check(name, n, [&] {
            lz_stream *st = nullptr;
            NEED(lz_stream_open(ctx, 0, pw, 7, &st) == LZ_OK);
            const int rc = lz_stream_update(st, in, n, out, nullptr);
            NEED(lz_stream_close(st) == LZ_OK);
            return rc;
        });
    }
    std::printf("refused launches: OK\n");
    return 0;
}
