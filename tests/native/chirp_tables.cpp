// Test program: the chirp convolution's tables (blu_tables in diag_fft.hip), run on the CPU with one thread per GPU
// thread of a workgroup.  The source is compiled as it stands, with the device's built-ins given here.  Checked
// for each length: every barrier is met by all threads of the workgroup at the same place in the code (anything else is
// undefined on the GPU), and the tables equal their definitions, summed directly in extended precision.
// Prints one line per length and "chirp tables: OK"; exit status 1 on a fault.
#include <hip/hip_runtime.h>

#include <barrier>
#include <cmath>
#include <complex>
#include <cstdio>
#include <thread>
#include <vector>

struct Idx { unsigned x = 0, y = 0, z = 0; };
static thread_local Idx threadIdx, blockIdx, gridDim;

constexpr int WG = 256;
static std::barrier<> meet(WG);
static int at_line[WG];
static bool g_split = false;  // written by thread 0 between the two waits

static void sync_at(int line) {
    at_line[threadIdx.x] = line;
    meet.arrive_and_wait();
    if (threadIdx.x == 0)
        for (int i = 1; i < WG; ++i)
            if (at_line[i] != at_line[0]) {
                if (!g_split) std::printf("thread 0 is at the barrier of line %d, thread %d at that of line %d\n", at_line[0], i, at_line[i]);
                g_split = true;
                break;
            }
    meet.arrive_and_wait();
}
#undef __syncthreads
#define __syncthreads() sync_at(__LINE__)

static void sincospi(double x, double *s, double *c) {
    const long double a = 3.14159265358979323846264338327950288L * x;
    *s = (double)sinl(a);
    *c = (double)cosl(a);
}

// parts of the file that are not run here
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) ((void)0)
#define __launch_bounds__(...)
#undef __shared__
#define __shared__
template <typename T> static T __shfl_xor(T v, int, int) { return v; }
template <typename A, typename C> static C mfma_stub(A, A, C c) { return c; }
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, ...) mfma_stub(a, b, c)
#define __builtin_amdgcn_wave_barrier() ((void)0)
#define __builtin_amdgcn_fence(...) ((void)0)

#include "../../paper_1201_3114_amd/csrc/diag_fft.hip"

namespace lz {
int diag_begin(lz_ctx *, hipStream_t, size_t, char **) { return 0; }
int diag_end(lz_ctx *, hipStream_t) { return 0; }
int fail(int code, const char *) { return code; }
int hip_fail(hipError_t, const char *) { return -1; }
namespace {
double2 fbuf[1];

typedef std::complex<long double> C;
C unit(long double turns) { return std::polar(1.0L, 6.28318530717958647692528676655900577L * turns); }

// A chirp value's error in eps = 2^-52: its argument e / N < 2 is rounded by at most 2^-53 (times pi), and cosine and
// sine by at most 2^-54 each (below 1).  A twiddle's argument is exact.
constexpr long double CHIRP = 3.1416L / 2 + 0.71L;

// The largest distance of a table's entries from their definitions, relative to eps and the entries' scale.
template <int R>
double check(uint32_t N) {
    using F = BluFft<R>;
    std::vector<double2> p(blu_entries(N) + 8, make_double2(7e77, 7e77)), lds(blu_table_lds(N) / sizeof(double2) + 8, make_double2(7e77, 7e77));
    constexpr uint32_t PARTS = 3;
    for (uint32_t part = 0; part < PARTS; ++part) {
        std::vector<std::thread> t;
        for (int i = 0; i < WG; ++i)
            t.emplace_back([&, i] {
                threadIdx.x = i;
                blu_tables<R>(p.data(), N, part, PARTS, lds.data());
            });
        for (auto &x : t) x.join();
    }
    auto kept = [](const std::vector<double2> &v) {
        for (size_t i = v.size() - 8; i < v.size(); ++i)
            if (v[i].x != 7e77 || v[i].y != 7e77) return false;
        return true;
    };
    if (!kept(p) || !kept(lds)) return INFINITY;  // written past its end
    const BluTab tab = blu_tab(p.data(), N);
    double worst = 0;
    auto cmp = [&](double2 got, C want, long double scale) {
        const double e = (double)(std::abs(C(got.x, got.y) - want) / scale / 2.220446049250313e-16L);
        if (!(e <= worst)) worst = e;
    };
    std::vector<C> c(N);
    for (uint32_t n = 0; n < N; ++n) {
        c[n] = unit(-(long double)(n * n % (2 * N)) / (2 * N));
        cmp(tab.c[n], c[n], CHIRP);
    }
    for (uint32_t i = 0; i < F::M; ++i) cmp(tab.ta[i], unit(-(long double)((i / F::T) * (i % F::T)) / F::M), 1);
    for (uint32_t i = 0; i < 16 * R; ++i) cmp(tab.tb[i], unit(-(long double)((i / 16) * (i % 16)) / F::T), 1);
    // the transform of b[m] = conj c[|m|], |m| < N, over M, and 1/M; scale: the 2-norm of b, times the bound of an FFT's
    // error (Higham, Accuracy and Stability of Numerical Algorithms, Theorem 24.2) and of the chirp's
    const long double scale = (7 * std::log2((double)F::M) + CHIRP) * std::sqrt(2.0L * N - 1) / F::M * std::sqrt((long double)F::M);
    for (uint32_t k = 0; k < F::M; k += F::M > 1024 ? 37 : 5) {
        C s = std::conj(c[0]);
        for (uint32_t n = 1; n < N; ++n) s += std::conj(c[n]) * (unit(-(long double)((uint64_t)n * k % F::M) / F::M) + unit((long double)((uint64_t)n * k % F::M) / F::M));
        cmp(tab.b[k], s / (long double)F::M, scale);
    }
    return worst;
}
}  // namespace
}  // namespace lz

int main() {
    bool ok = true;
    for (uint32_t N : {80u, 83u, 251u, 256u, 257u, 509u, 521u, 1009u, 1031u, 2039u}) {
        double e = 0;
        switch (lz::blu_r(N)) {
            case 2: e = lz::check<2>(N); break;
            case 4: e = lz::check<4>(N); break;
            case 8: e = lz::check<8>(N); break;
            default: e = lz::check<16>(N); break;
        }
        std::printf("length %u: error %.3g of its bound\n", N, e);
        ok = ok && e <= 1.0 && !g_split;
    }
    std::printf("%s\n", ok ? "chirp tables: OK" : "chirp tables: FAULT");
    return ok ? 0 : 1;
}
