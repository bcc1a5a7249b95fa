// Test program: fix_range_part of diag_lags.hip (the sum of the first or last bytes of a sequence, thread by thread) on the CPU,
// for short sequences at every alignment, laid against unreadable pages on both sides.  LAG_ENDS_PART names a file that
// holds the function as it stands in the source.  A read out of range ends the program, a wrong sum is printed.
#include <hip/hip_runtime.h>
#include <sys/mman.h>
#include <unistd.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>

struct Idx { unsigned x = 0; };
static Idx threadIdx;
constexpr int DIAG_WG = 256;

static uint32_t udot4(uint32_t a, uint32_t b, uint32_t c, bool) {
    for (int i = 0; i < 4; ++i) c += ((a >> (8 * i)) & 0xFF) * ((b >> (8 * i)) & 0xFF);
    return c;
}
#define __builtin_amdgcn_udot4 udot4

namespace {
#include LAG_ENDS_PART

unsigned long long whole(const uint8_t *data, uint64_t lo, uint64_t hi) {
    unsigned long long s = 0;
    for (int t = 0; t < DIAG_WG; ++t) {
        threadIdx.x = t;
        s += fix_range_part(data, lo, hi);
    }
    return s;
}
}  // namespace

int main() {
    const size_t page = (size_t)sysconf(_SC_PAGESIZE), body = 10 * page;
    uint8_t *map = (uint8_t *)mmap(nullptr, body + 2 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (map == (uint8_t *)MAP_FAILED) return 2;
    mprotect(map, page, PROT_NONE);
    mprotect(map + page + body, page, PROT_NONE);
    uint8_t *first = map + page;
    for (size_t i = 0; i < body; ++i) first[i] = (uint8_t)(1 + i * 37 % 255);
    long cases = 0;
    for (uint64_t n : {0, 1, 2, 3, 5, 8, 9, 14, 15, 16, 17, 31, 32, 33, 47, 100, 257, 5000, 20000})
        for (int at = 0; at < 34; ++at) {
            // by the first page for at < 17, against the last for the others
            const uint8_t *data = at < 17 ? first + at : first + body - n - (at - 17);
            for (uint64_t m : {(uint64_t)0, (uint64_t)1, (uint64_t)2, (uint64_t)7, (uint64_t)15, (uint64_t)16, (uint64_t)256, (uint64_t)4864, n}) {
                if (m > n) continue;
                for (int end = 0; end < 2; ++end) {
                    const uint64_t lo = end ? n - m : 0, hi = end ? n : m;
                    unsigned long long want = 0;
                    for (uint64_t i = lo; i < hi; ++i) want += data[i];
                    const unsigned long long got = whole(data, lo, hi);
                    ++cases;
                    if (got != want) {
                        std::printf("n %llu at %d: bytes %llu to %llu give %llu, not %llu\n", (unsigned long long)n, at,
                                    (unsigned long long)lo, (unsigned long long)hi, got, want);
                        return 1;
                    }
                }
            }
        }
    std::printf("%ld cases\nlag ends: OK\n", cases);
    return 0;
}
