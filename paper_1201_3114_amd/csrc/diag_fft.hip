// The 2-D analyses of Section 4 for a byte matrix (a text or an image laid out row by row) as
// GPU kernels: the Fourier power spectrum and the circular autocorrelation matrix, in binary64.
// The 2-D transforms run as FFTs for sides with no prime factor above 5, as FFT convolutions (Bluestein)
// for other sides from 80 to 2048, and as binary64 matrix products on the matrix cores otherwise.
#include "diag_common.h"

#include <type_traits>

namespace lz {
namespace {

// ---- 2-D discrete Fourier transform as two passes ----------------------------------------
//
// One pass applies the N-point DFT along the rows index of an N x M matrix and
// writes the result transposed:  dst[c][r] = sum_k e^{sign 2 pi i r k / N} src[k][c].
// Two passes (first along the H rows of the H x W image, then along its W
// columns) give the 2-D DFT in natural layout.  Every size is allowed (no
// power-of-two restriction); the twiddle index r k mod N is kept exact in
// integers, so every twiddle is one table entry.

constexpr int DFT_T = 64;  // output tile edge (r and c)
constexpr int DFT_KS32 = 32, DFT_KS64 = 16;  // terms per LDS stage for 32- and 64-row tiles

// (cos 2 pi j / N, sin 2 pi j / N)
__device__ __forceinline__ double2 twiddle_of(uint32_t j, uint32_t N) {
    double s, c;
    sincospi(2.0 * (double)j / (double)N, &s, &c);
    return make_double2(c, s);
}

// an input value as a complex number; bytes less their middle value
__device__ __forceinline__ double2 dft_value(uint8_t v, double mid) { return make_double2((double)v - mid, 0.0); }
__device__ __forceinline__ double2 dft_value(double v, double) { return make_double2(v, 0.0); }
__device__ __forceinline__ double2 dft_value(double2 v, double) { return v; }

// The pass runs on the matrix cores: binary64 MFMA 16x16x4 (v_mfma_f64_16x16x4f64), operand
// layout: lane i holds A[i % 16][i / 16] and B[i / 16][i % 16] of the 16x4 and 4x16 operands,
// and D[4 j + i / 16][i % 16] in its j-th accumulator.  A complex product takes four real
// products: re += wr xr - wi xi, im += wr xi + wi xr.  The inputs and twiddles of the next
// k stage (16 or 32 terms) are loaded into registers while the current stage computes; the loads are
// unconditional, from valid addresses, so nothing waits for them before the stage's products,
// and out-of-range entries are zeroed when stored to LDS.
typedef double v4d __attribute__((ext_vector_type(4)));

// What a pass writes for output (column c, index r) of its transforms, row-major in its
// M x nout output: the complex value, |Z|^2, |Z|^2 with the zero frequency (c = r = 0 of the
// second pass) set to 0, or Re Z / den (the normalised autocorrelation; NaN when den is).
// A real matrix (h rows) has a Hermitian 2-D transform, Z[h - k1][w - k2] = conj Z[k1][k2]
// (indices mod h and w), so a first pass over real columns keeps only indices r < nout =
// h/2 + 1 of each column's transform, the second pass transforms those h/2 + 1 columns, and
// its real results (|Z|^2, or Re Z of an even real matrix's transform) are written twice:
// row c, and, as row h - c with k2 -> w - k2, each row the pass does not compute itself
// (mirror = h; 0 writes no mirror rows).
// The sums S1 = sum x and S2 = sum x^2 over the bytes come from workgroups of their own in the launch that
// makes the tables (tables_kernel), one pair of words per workgroup, exact (S1 < 2^32 and S2 < 2^40 for at
// most 2^24 bytes).  They give the autocorrelation matrix's denominator n S2 - S1^2 in the last pass (NaN
// when n S2 = S1^2, that is when every byte is equal), and the mean: a first pass transforms x - m, m the
// mean to the nearest whole number, so the subtraction is exact, the mean, mostly the largest part of the
// input, makes no rounding errors, and the spectrum's second pass adds m h w to the zero frequency.
constexpr uint32_t SUM_WGS = 256;  // pairs, at most
enum : int { EPI_COMPLEX = 0, EPI_POWER = 1, EPI_POWER_NODC = 2, EPI_ACF = 3 };
struct Sums {
    const unsigned long long *p;  // S1, S2 of workgroup 0, 1, ... (NULL: none, m = 0)
    uint32_t wgs;
    uint64_t n;                   // bytes of the matrix
};
struct PassOut {
    double2 *z;
    double *p;
    uint32_t nout;
    uint32_t mirror;
    Sums sums;
    double den;               // EPI_ACF: set by the kernel from the sums
    double dc;                // EPI_POWER: m h w, set by the kernel from the sums
};

// S1 and S2; every lane of a wave calls it and has the result.
__device__ __forceinline__ void total_sums(const Sums &q, unsigned long long &s1, unsigned long long &s2) {
    s1 = s2 = 0;
    for (uint32_t i = threadIdx.x & 63; i < q.wgs; i += 64) {
        s1 += q.p[2 * i];
        s2 += q.p[2 * i + 1];
    }
    for (int k = 32; k > 0; k >>= 1) {
        s1 += __shfl_xor(s1, k, 64);
        s2 += __shfl_xor(s2, k, 64);
    }
}

// m: the mean byte to the nearest whole number.
__device__ __forceinline__ double byte_mid(const Sums &q) {
    if (!q.p) return 0.0;
    unsigned long long s1, s2;
    total_sums(q, s1, s2);
    return rint((double)s1 / (double)q.n);
}

// What a pass's store needs of the sums.
template <int E>
__device__ __forceinline__ void pass_sums(PassOut &o) {
    if constexpr (E == EPI_ACF) {
        unsigned long long s1, s2;
        total_sums(o.sums, s1, s2);
        const unsigned long long d = o.sums.n * s2 - s1 * s1;  // n <= 2^24 keeps both products below 2^64
        o.den = d == 0 ? __builtin_nan("") : (double)d;
    } else if constexpr (E == EPI_POWER) {
        o.dc = byte_mid(o.sums) * (double)o.sums.n;
    }
}

template <int E>
__device__ __forceinline__ void pass_store(const PassOut &o, uint32_t c, uint32_t r, uint32_t N, uint32_t M,
                                           double re, double im) {
    if (r >= o.nout) return;
    const size_t i = (size_t)c * o.nout + r;
    if constexpr (E == EPI_COMPLEX) {
        o.z[i] = make_double2(re, im);
    } else {
        double v;
        if constexpr (E == EPI_ACF) {
            const double d = o.den;
            v = d != d ? d : re / d;
        } else {
            if (E == EPI_POWER && c == 0 && r == 0) re += o.dc;
            v = (E == EPI_POWER_NODC && c == 0 && r == 0) ? 0.0 : re * re + im * im;
        }
        o.p[i] = v;
        // the real outputs keep whole rows (nout = N)
        if (o.mirror && c != 0 && o.mirror - c >= M) o.p[(size_t)(o.mirror - c) * N + (r ? N - r : 0)] = v;
    }
}

template <typename In, int E, int TR, int KS>
__global__ __launch_bounds__(DIAG_WG) void dft_pass_kernel(const In *src, uint32_t N, uint32_t M, const double2 *tw,
                                                            double sign, PassOut dst) {
    pass_sums<E>(dst);
    // Workgroups are dealt to the 8 XCDs in turn: when the tiles divide evenly, those sharing an
    // input column tile go to one XCD, whose L2 then reads those columns from HBM once.
    const uint32_t nt = gridDim.x * gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
    const uint32_t tix = nt % 8 == 0 ? (lin % 8) * (nt / 8) + lin / 8 : lin;
    const uint32_t rt = tix % gridDim.x, ct = tix / gridDim.x;  // row tile, column tile
    const double mid = std::is_same_v<In, uint8_t> ? byte_mid(dst.sums) : 0.0;
    // TR x 64 outputs per workgroup: with TR = 64 each wave takes a 32 x 32 block as 2 x 2 tiles of
    // 16 x 16, with TR = 32 (grids that would not fill the chip) a 32 x 16 block as 2 x 1 tiles.
    // A real input (bytes or doubles) has no imaginary part: two of the four products are skipped.
    // KS terms per LDS stage: the loads of the next stage are in flight during this one's products.
    static_assert(TR == 64 || TR == 32, "tile height");
    static_assert(KS % 4 == 0 && (TR * KS) % DIAG_WG == 0, "whole rows of the stage per thread");
    constexpr int QX = KS / 4;                       // input rows each thread stages per k stage
    constexpr int WC = TR == 64 ? 2 : 4;             // waves across the tile's columns
    constexpr int TB = 4 / WC;                       // column tiles per wave
    constexpr bool REAL = !std::is_same_v<In, double2>;
    constexpr int TWQ = TR * KS / DIAG_WG;           // twiddles each thread stages per k stage
    __shared__ double2 s_src[KS][DFT_T];  // [k][c]
    __shared__ double2 s_tw[KS][TR];      // [k][r]
    const uint32_t r0 = rt * TR, c0 = ct * DFT_T;
    const uint32_t lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const uint32_t wr = (wave / WC) * 32, wc = (wave % WC) * (16 * TB);
    const uint32_t li = lane % 16, lk = lane / 16;
    // staging: column cc of the input tile for k rows kq + 4q; twiddle row tr_s for k rows kt + (KS/TWQ) q
    const uint32_t cc = threadIdx.x % DFT_T, kq = threadIdx.x / DFT_T;
    const uint32_t tr_s = threadIdx.x % TR, kt = threadIdx.x / TR;
    const uint32_t rs = r0 + tr_s;
    const uint32_t rmod = rs < N ? rs : 0;
    const uint32_t cs = c0 + cc < M ? c0 + cc : M - 1;
    uint32_t off[TWQ];
    for (int q = 0; q < TWQ; ++q) off[q] = (uint32_t)(((uint64_t)rmod * (kt + (KS / TWQ) * q)) % N);
    const uint32_t step = (uint32_t)(((uint64_t)rmod * KS) % N);
    uint32_t base = 0;
    In nx[QX];
    double2 nw[TWQ];
    auto fetch = [&](uint32_t k0) {
        for (int q = 0; q < QX; ++q) {
            const uint32_t k = k0 + kq + 4 * q;
            nx[q] = src[(size_t)(k < N ? k : N - 1) * M + cs];
        }
        for (int q = 0; q < TWQ; ++q) {
            uint32_t j = base + off[q];
            if (j >= N) j -= N;
            nw[q] = tw[j];
        }
        base += step;
        if (base >= N) base -= N;
    };
    v4d re[2][TB], im[2][TB];
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < TB; ++b) re[a][b] = im[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
    fetch(0);
    for (uint32_t k0 = 0; k0 < N; k0 += KS) {
        for (int q = 0; q < QX; ++q) {
            const uint32_t k = k0 + kq + 4 * q;
            const bool in = k < N && c0 + cc < M;
            s_src[kq + 4 * q][cc] = in ? dft_value(nx[q], mid) : make_double2(0.0, 0.0);
        }
        for (int q = 0; q < TWQ; ++q) {
            const uint32_t kk = kt + (KS / TWQ) * q, k = k0 + kk;
            s_tw[kk][tr_s] = (k < N && rs < N) ? make_double2(nw[q].x, sign * nw[q].y) : make_double2(0.0, 0.0);
        }
        __syncthreads();
        if (k0 + KS < N) fetch(k0 + KS);
#pragma unroll
        for (int k4 = 0; k4 < KS / 4; ++k4) {
            const int k = 4 * k4 + (int)lk;
            double2 w[2], x[TB];
            for (int t = 0; t < 2; ++t) w[t] = s_tw[k][wr + 16 * t + li];
            for (int t = 0; t < TB; ++t) x[t] = s_src[k][wc + 16 * t + li];
            for (int a = 0; a < 2; ++a)
                for (int b = 0; b < TB; ++b) {
                    re[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[a].x, x[b].x, re[a][b], 0, 0, 0);
                    if constexpr (!REAL) {
                        re[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-w[a].y, x[b].y, re[a][b], 0, 0, 0);
                        im[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[a].x, x[b].y, im[a][b], 0, 0, 0);
                    }
                    im[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[a].y, x[b].x, im[a][b], 0, 0, 0);
                }
        }
        __syncthreads();
    }
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < TB; ++b)
            for (int j = 0; j < 4; ++j) {
                const uint32_t r = r0 + wr + 16 * a + 4 * j + lk, c = c0 + wc + 16 * b + li;
                if (r < N && c < M) pass_store<E>(dst, c, r, N, M, re[a][b][j], im[a][b][j]);
            }
}

// ---- the same pass by FFT, for power-of-two lengths -------------------------------------
//
// For N = 2^p <= FFT_MAX the pass uses Stockham autosort stages (the self-sorting
// FFT): with stride s and n = N / s, a radix-r stage reads the r values
// x[q + s (j + l n / r)], l < r, takes their r-point DFT, multiplies output k by
// W_n^{j k} and writes it to x[q + s (r j + k)], so the result ends in natural
// order.  Radix-4 stages, after one radix-2 stage when p is odd.  A workgroup
// transforms C adjacent columns in LDS: each input row is read as C contiguous
// elements and each output row (one column's transform) is written contiguously.
// Each workgroup computes W^b, b < N/4 (W = e^{sign 2 pi i / N}), into LDS while its
// input loads are in flight; the stages' other twiddles follow exactly, as
// W^{a N/4 + b} = (sign i)^a W^b.  About 2.1 p flops per value instead of the
// direct pass's 8 N.
constexpr uint32_t FFT_MAX = 4096;
constexpr uint32_t FFT_PP_MAX = 1024;             // two LDS copies of the columns up to this length (36 KB)
constexpr uint32_t FFT_WG_ELEMS = 1024;           // complex values per workgroup when N <= 1024 (16 KB of LDS)
constexpr int FFT_EPT = FFT_MAX / DIAG_WG;        // values per thread, at most
constexpr int FFT_B2 = FFT_MAX / 2 / DIAG_WG;     // radix-2 butterflies per thread, at most
constexpr int FFT_B4 = FFT_MAX / 4 / DIAG_WG;     // radix-4 butterflies per thread per stage, at most

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 w) {
    return make_double2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}

__host__ __device__ constexpr uint32_t fft_twiddles(uint32_t N) { return N < 4 ? 1 : N / 4; }

// W^j for j < 3N/4 from the quarter table q[b] = W^b: multiplying by W^{N/4} = sign i is exact.
__device__ __forceinline__ double2 fft_twiddle(const double2 *q, uint32_t j, uint32_t logN, double sign) {
    if (logN < 2) return make_double2(1.0, 0.0);  // N <= 2 uses j = 0 only
    const double2 w = q[j & ((1u << (logN - 2)) - 1)];
    switch (j >> (logN - 2)) {
        case 0: return w;
        case 1: return make_double2(-sign * w.y, sign * w.x);
        default: return make_double2(-w.x, -w.y);
    }
}

template <typename In, int E>
__global__ __launch_bounds__(DIAG_WG) void fft_pass_kernel(const In *src, uint32_t N, uint32_t M, uint32_t logN,
                                                            uint32_t C, double sign, PassOut dst) {
    pass_sums<E>(dst);
    // C columns of N values (twice when N <= FFT_PP_MAX: each stage reads one copy and writes the
    // other, so it needs one barrier instead of two), then the twiddles
    extern __shared__ double2 fbuf[];
    const bool pp = N <= FFT_PP_MAX;
    double2 *cur = fbuf, *nxt = fbuf + (pp ? (size_t)C * N : 0);
    double2 *ftw = fbuf + (size_t)(pp ? 2 : 1) * C * N;
    // consecutive column groups on the same XCD (workgroups are dealt to the 8 XCDs in turn),
    // so the partly shared cache lines of neighbouring groups meet in one L2
    uint32_t g = blockIdx.x;
    if (gridDim.x % 8 == 0) g = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const uint32_t c0 = g * C;
    if (c0 >= M) return;  // a workgroup of the padding (the grid is a multiple of 8)
    const uint32_t cols = M - c0 < C ? M - c0 : C;
    const uint32_t total = cols * N;
    {
        // all of a thread's loads are issued before the first is stored, and the twiddles
        // (the values the table kernel computes: sincospi of 2j / N) are made meanwhile
        In v[FFT_EPT];
#pragma unroll
        for (int i = 0; i < FFT_EPT; ++i) {
            const uint32_t e = threadIdx.x + i * DIAG_WG;
            if (e < total) {
                const uint32_t k = e / cols, cl = e - k * cols;
                v[i] = src[(size_t)k * M + c0 + cl];
            }
        }
        for (uint32_t j = threadIdx.x; j < fft_twiddles(N); j += DIAG_WG) {
            double sn, cs;
            sincospi(2.0 * (double)j / (double)N, &sn, &cs);
            ftw[j] = make_double2(cs, sign * sn);
        }
        const double mid = std::is_same_v<In, uint8_t> ? byte_mid(dst.sums) : 0.0;
#pragma unroll
        for (int i = 0; i < FFT_EPT; ++i) {
            const uint32_t e = threadIdx.x + i * DIAG_WG;
            if (e < total) {
                const uint32_t k = e / cols, cl = e - k * cols;
                cur[cl * N + k] = dft_value(v[i], mid);
            }
        }
    }
    __syncthreads();
    uint32_t st = 0;  // log2 of the stride s
    if (logN & 1) {
        // radix-2 stage, s = 1: x[j], x[j + N/2] -> x[2j], x[2j + 1]
        const uint32_t half = N >> 1, nb = cols * half;
        double2 a[FFT_B2], b[FFT_B2];
#pragma unroll
        for (int i = 0; i < FFT_B2; ++i) {
            const uint32_t u = threadIdx.x + i * DIAG_WG;
            if (u < nb) {
                const double2 *x = cur + (u >> (logN - 1)) * N;
                const uint32_t j = u & (half - 1);
                a[i] = x[j];
                b[i] = x[j + half];
            }
        }
        if (!pp) __syncthreads();
#pragma unroll
        for (int i = 0; i < FFT_B2; ++i) {
            const uint32_t u = threadIdx.x + i * DIAG_WG;
            if (u < nb) {
                double2 *x = nxt + (u >> (logN - 1)) * N;
                const uint32_t j = u & (half - 1);
                x[2 * j] = cadd(a[i], b[i]);
                x[2 * j + 1] = cmul(csub(a[i], b[i]), fft_twiddle(ftw, j, logN, sign));
            }
        }
        __syncthreads();
        double2 *t = cur;
        cur = nxt;
        nxt = t;
        st = 1;
    }
    const uint32_t quarter = N >> 2, nb4 = cols * quarter;
    for (; st < logN; st += 2) {
        const uint32_t s = 1u << st, m = N >> (st + 2);
        double2 a[FFT_B4][4];
#pragma unroll
        for (int i = 0; i < FFT_B4; ++i) {
            const uint32_t u = threadIdx.x + i * DIAG_WG;
            if (u < nb4) {
                const double2 *x = cur + (u >> (logN - 2)) * N;
                const uint32_t t = u & (quarter - 1), q = t & (s - 1), j = t >> st;
#pragma unroll
                for (int l = 0; l < 4; ++l) a[i][l] = x[q + s * (j + l * m)];
            }
        }
        if (!pp) __syncthreads();
#pragma unroll
        for (int i = 0; i < FFT_B4; ++i) {
            const uint32_t u = threadIdx.x + i * DIAG_WG;
            if (u < nb4) {
                double2 *x = nxt + (u >> (logN - 2)) * N;
                const uint32_t t = u & (quarter - 1), q = t & (s - 1), j = t >> st;
                const double2 t0 = cadd(a[i][0], a[i][2]), t1 = csub(a[i][0], a[i][2]);
                const double2 t2 = cadd(a[i][1], a[i][3]), t3 = csub(a[i][1], a[i][3]);
                const double2 rt3 = make_double2(-sign * t3.y, sign * t3.x);  // W_4 t3, W_4 = sign i
                const uint32_t w = t - q;                                    // j s: W_n^{j k} = table[j s k]
                x[q + s * (4 * j)] = cadd(t0, t2);
                x[q + s * (4 * j + 1)] = cmul(cadd(t1, rt3), fft_twiddle(ftw, w, logN, sign));
                x[q + s * (4 * j + 2)] = cmul(csub(t0, t2), fft_twiddle(ftw, 2 * w, logN, sign));
                x[q + s * (4 * j + 3)] = cmul(csub(t1, rt3), fft_twiddle(ftw, 3 * w, logN, sign));
            }
        }
        __syncthreads();
        double2 *t = cur;
        cur = nxt;
        nxt = t;
    }
    for (uint32_t e = threadIdx.x; e < total; e += DIAG_WG) {
        const double2 v = cur[e];
        pass_store<E>(dst, c0 + (e >> logN), e & (N - 1), N, M, v.x, v.y);
    }
}

// ---- the same pass by mixed-radix FFT, for lengths 2^a 3^b 5^c --------------------------
//
// ---- 1024-point pass: one wave per column, three register stages -----------------------
//
// With n = t + 64 j and k = k1 + 16 k2 (t, k2 < 64; j, k1 < 16),
//   X[k1 + 16 k2] = sum_t W_64^{t k2} [W_1024^{t k1} sum_j x[t + 64 j] W_16^{j k1}],
// and the 64-point DFTs over t split again as t = a + 4 b, k2 = c + 16 d (a, d < 4; b, c < 16):
//   Y[c + 16 d] = sum_a W_4^{a d} [W_64^{a c} sum_b y[a + 4 b] W_16^{b c}].
// Lane t of a column's wave loads x[t + 64 j] (16 values), takes their 16-point DFT in registers
// and the twiddles W_1024^{t k1}; through LDS, lane (k1, a) = (t / 4, t % 4) takes the 16 values
// y[a + 4 b] of its k1, their 16-point DFT and the twiddles W_64^{a c}; through LDS again, each
// lane takes four 4-point DFTs over a and stores X[k1 + 16 c + 256 d], 64 consecutive outputs per
// store.  The LDS row strides (68 and 258 entries of 16 bytes) put the 8 lanes of each 128-byte
// LDS cycle on distinct banks in every exchange.  The workgroup makes the quarter twiddle table
// W^b, b < 256, while its loads are in flight.  A 16-point DFT is 4 x 4: 4-point DFTs, the
// twiddles W_16^{n2 k1}, 4-point DFTs.
constexpr uint32_t FFT1K = 1024;
constexpr int FFT1K_COLS = DIAG_WG / 64;  // columns per workgroup, one per wave
constexpr int FFT1K_S1 = 68;              // LDS row stride of the stage-1 output (rows k1)
constexpr int FFT1K_S2 = 258;             // LDS row stride of the stage-2 output (rows a)
constexpr int FFT1K_WAVE = 16 * FFT1K_S1; // LDS entries per wave (the stage-2 output fits in them)

static_assert(DIAG_WG == FFT1K / 4, "one quarter-table entry per thread");

// Orders a wave's LDS accesses before and after this point for the compiler; the wave's own
// LDS operations complete in order, so its lanes then see each other's stores.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__host__ __device__ constexpr size_t fft1k_lds() { return ((size_t)FFT1K_COLS * FFT1K_WAVE + FFT1K / 4) * 16; }

// z (sign i)^q
__device__ __forceinline__ double2 rot_q(double2 z, uint32_t q, double sign) {
    switch (q & 3) {
        case 0: return z;
        case 1: return make_double2(-sign * z.y, sign * z.x);
        case 2: return make_double2(-z.x, -z.y);
        default: return make_double2(sign * z.y, -sign * z.x);
    }
}

// W^j, j < 1024, from the quarter table q[b] = W^b (b < 256)
__device__ __forceinline__ double2 tw1k(const double2 *q, uint32_t j, double sign) {
    return rot_q(q[j & 255], j >> 8, sign);
}

__device__ __forceinline__ void dft4(double2 &a0, double2 &a1, double2 &a2, double2 &a3, double sign) {
    const double2 t0 = cadd(a0, a2), t1 = csub(a0, a2), t2 = cadd(a1, a3), t3 = rot_q(csub(a1, a3), 1, sign);
    a0 = cadd(t0, t2);
    a1 = cadd(t1, t3);
    a2 = csub(t0, t2);
    a3 = csub(t1, t3);
}

// v[k] <- sum_n v[n] W_16^{n k}, W_16 = e^{sign 2 pi i / 16}
__device__ __forceinline__ void dft16(double2 (&v)[16], double sign) {
    constexpr double C1 = 0.92387953251128674;  // cos(pi / 8)
    constexpr double S1 = 0.38268343236508977;  // sin(pi / 8)
    constexpr double R2 = 0.70710678118654752;  // cos(pi / 4)
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) dft4(v[n2], v[4 + n2], v[8 + n2], v[12 + n2], sign);
    // v[4 k1 + n2] now holds A[n2][k1]; twiddles W_16^{n2 k1}
    v[5] = cmul(v[5], make_double2(C1, sign * S1));     // n2 = 1, k1 = 1
    v[9] = cmul(v[9], make_double2(R2, sign * R2));     // 1, 2
    v[13] = cmul(v[13], make_double2(S1, sign * C1));   // 1, 3
    v[6] = cmul(v[6], make_double2(R2, sign * R2));     // 2, 1
    v[10] = rot_q(v[10], 1, sign);                      // 2, 2
    v[14] = cmul(v[14], make_double2(-R2, sign * R2));  // 2, 3
    v[7] = cmul(v[7], make_double2(S1, sign * C1));     // 3, 1
    v[11] = cmul(v[11], make_double2(-R2, sign * R2));  // 3, 2
    v[15] = cmul(v[15], make_double2(-C1, -sign * S1)); // 3, 3
    double2 u[16];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
        double2 a0 = v[4 * k1], a1 = v[4 * k1 + 1], a2 = v[4 * k1 + 2], a3 = v[4 * k1 + 3];
        dft4(a0, a1, a2, a3, sign);
        u[k1] = a0;
        u[k1 + 4] = a1;
        u[k1 + 8] = a2;
        u[k1 + 12] = a3;
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = u[k];
}

template <typename In, int E>
__global__ __launch_bounds__(DIAG_WG) void fft1k_pass_kernel(const In *src, uint32_t M, double sign, PassOut dst) {
    pass_sums<E>(dst);
    extern __shared__ double2 fbuf[];
    const uint32_t lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    double2 *L = fbuf + (size_t)wave * FFT1K_WAVE;
    double2 *q = fbuf + (size_t)FFT1K_COLS * FFT1K_WAVE;
    // consecutive column groups on the same XCD (workgroups are dealt to the 8 XCDs in turn)
    uint32_t g = blockIdx.x;
    if (gridDim.x % 8 == 0) g = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const uint32_t col = g * FFT1K_COLS + wave;
    const bool live = col < M;
    In x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (live) x[j] = src[(size_t)(lane + 64 * j) * M + col];
    {
        double sn, cs;
        sincospi(2.0 * (double)threadIdx.x / (double)FFT1K, &sn, &cs);
        q[threadIdx.x] = make_double2(cs, sign * sn);
    }
    const double mid = std::is_same_v<In, uint8_t> ? byte_mid(dst.sums) : 0.0;
    __syncthreads();
    if (!live) return;  // the whole wave
    double2 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = dft_value(x[j], mid);
    // stage 1: 16-point DFT over j, twiddles W^{t k1}
    dft16(v, sign);
#pragma unroll
    for (int k1 = 0; k1 < 16; ++k1) L[k1 * FFT1K_S1 + lane] = k1 ? cmul(v[k1], tw1k(q, lane * k1, sign)) : v[0];
    wave_fence();
    // stage 2: lane (k1, a) takes y[a + 4 b][k1], a 16-point DFT over b, twiddles W_64^{a c}
    const uint32_t k1 = lane >> 2, a = lane & 3;
#pragma unroll
    for (int b = 0; b < 16; ++b) v[b] = L[k1 * FFT1K_S1 + a + 4 * b];
    wave_fence();
    dft16(v, sign);
#pragma unroll
    for (int c = 0; c < 16; ++c)
        L[a * FFT1K_S2 + c * 16 + k1] = (a && c) ? cmul(v[c], tw1k(q, 16 * a * c, sign)) : v[c];
    wave_fence();
    // stage 3: 4-point DFTs over a of pairs p = 16 c + k1 = 64 i + lane; X[p + 256 d]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t p = 64 * i + lane;
        double2 a0 = L[p], a1 = L[FFT1K_S2 + p], a2 = L[2 * FFT1K_S2 + p], a3 = L[3 * FFT1K_S2 + p];
        dft4(a0, a1, a2, a3, sign);
        pass_store<E>(dst, col, p, FFT1K, M, a0.x, a0.y);
        pass_store<E>(dst, col, p + 256, FFT1K, M, a1.x, a1.y);
        pass_store<E>(dst, col, p + 512, FFT1K, M, a2.x, a2.y);
        pass_store<E>(dst, col, p + 768, FFT1K, M, a3.x, a3.y);
    }
}

// ---- two real columns as one complex column ---------------------------------------------
//
// The mixed-radix and the chirp pass over real columns (bytes, or the inverse passes' real spectrum) transform
// z = x1 + i x2 for columns 2p and 2p + 1; X1 and X2 are the even and odd parts of Z, of which only the indices
// up to N/2 are kept.  That halves the transforms: 1000 x 1000 takes 41 and 76 us (spectrum and correlation
// matrix, calls back to back), 52 and 104 with a transform per column.  The two columns share their rounding errors; without the mean
// (see Sums) these are no larger than they were with it in a transform per column.
template <typename In>
constexpr uint32_t per_transform() { return std::is_same_v<In, double2> ? 1 : 2; }

template <typename In>
struct PackIn { In a, b; };
template <>
struct PackIn<double2> { double2 a; };

// The input of transform p at row k of the N x M matrix src.
template <typename In>
__device__ __forceinline__ PackIn<In> pack_load(const In *src, uint32_t k, uint32_t p, uint32_t M) {
    if constexpr (std::is_same_v<In, double2>) {
        return PackIn<In>{src[(size_t)k * M + p]};
    } else {
        const In *q = src + (size_t)k * M + 2 * p;
        PackIn<In> v;
        if (2 * p + 1 < M) {
            __builtin_memcpy(&v, q, sizeof v);  // one load of both
        } else {
            v.a = *q;
            v.b = In{};
        }
        return v;
    }
}

template <typename In>
__device__ __forceinline__ double2 pack_value(const PackIn<In> &v, double mid) {
    if constexpr (std::is_same_v<In, double2>) return v.a;
    else return make_double2((double)v.a - mid, (double)v.b - mid);  // mid = 0 but for bytes
}

// Indices k and N - k of a transform of columns c and c + 1 -> index k of both.
template <int E>
__device__ __forceinline__ void pair_store(const PassOut &o, uint32_t c, uint32_t k, uint32_t N, uint32_t M, double2 a,
                                           double2 b) {
    pass_store<E>(o, c, k, N, M, 0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    if (c + 1 < M) pass_store<E>(o, c + 1, k, N, M, 0.5 * (a.y + b.y), 0.5 * (b.x - a.x));
}

// Lengths N <= FFT_MAX whose only prime factors are 2, 3 and 5 (and that are not
// powers of two) run as Stockham stages of radix 5, 3, 4 and 2 in turn (the radix
// of each stage in FftPlan).  A radix-R stage with stride s, n = N / s, reads
// x[q + s (j + l n/R)] for l < R, takes their R-point DFT (radix 2 and 4 in
// their exact +-1, +-i form, radix 3 and 5 with W_R^p = W_N^{p N/R} from the
// table), multiplies output k by W_n^{jk} = W_N^{j s k} and writes it to
// x[q + s (R j + k)].  The N-entry table (the twiddle kernel's, sign applied) is
// copied into LDS beside the data; the rest is as in fft_pass_kernel.
struct FftPlan {
    uint32_t nst;
    uint8_t rad[16];
};

template <int R>
__device__ __forceinline__ void mixed_stage(double2 *fbuf, const double2 *ftw, uint32_t N, uint32_t cols,
                                            uint32_t s, double sign) {
    constexpr int BPT = (int)((FFT_MAX / R + DIAG_WG - 1) / DIAG_WG);
    const uint32_t nr = N / R, m = nr / s, nb = cols * nr, step = N / R;
    double2 a[BPT][R];
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        const uint32_t u = threadIdx.x + i * DIAG_WG;
        if (u < nb) {
            const uint32_t cl = u / nr, t = u - cl * nr, j = t / s, q = t - j * s;
            const double2 *x = fbuf + (size_t)cl * N;
#pragma unroll
            for (int l = 0; l < R; ++l) a[i][l] = x[q + s * (j + l * m)];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        const uint32_t u = threadIdx.x + i * DIAG_WG;
        if (u < nb) {
            const uint32_t cl = u / nr, t = u - cl * nr, j = t / s, q = t - j * s;
            double2 y[R];
            if constexpr (R == 2) {
                y[0] = cadd(a[i][0], a[i][1]);
                y[1] = csub(a[i][0], a[i][1]);
            } else if constexpr (R == 4) {
                const double2 t0 = cadd(a[i][0], a[i][2]), t1 = csub(a[i][0], a[i][2]);
                const double2 t2 = cadd(a[i][1], a[i][3]), t3 = csub(a[i][1], a[i][3]);
                const double2 rt3 = make_double2(-sign * t3.y, sign * t3.x);  // W_4 t3, W_4 = sign i
                y[0] = cadd(t0, t2);
                y[1] = cadd(t1, rt3);
                y[2] = csub(t0, t2);
                y[3] = csub(t1, rt3);
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    double2 acc = a[i][0];
#pragma unroll
                    for (int l = 1; l < R; ++l)
                        acc = k == 0 ? cadd(acc, a[i][l]) : cadd(acc, cmul(a[i][l], ftw[((l * k) % R) * step]));
                    y[k] = acc;
                }
            }
            double2 *x = fbuf + (size_t)cl * N;
            x[q + s * (R * j)] = y[0];
#pragma unroll
            for (int k = 1; k < R; ++k) x[q + s * (R * j + k)] = cmul(y[k], ftw[j * s * k]);
        }
    }
    __syncthreads();
}

template <typename In, int E>
__global__ __launch_bounds__(DIAG_WG) void fft_mixed_pass_kernel(const In *src, uint32_t N, uint32_t M, uint32_t C,
                                                                  FftPlan plan, const double2 *tw, double sign,
                                                                  PassOut dst) {
    pass_sums<E>(dst);
    extern __shared__ double2 fbuf[];  // C transforms of N values, then the N twiddles
    double2 *ftw = fbuf + (size_t)C * N;
    uint32_t g = blockIdx.x;
    if (gridDim.x % 8 == 0) g = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const uint32_t c0 = g * C, MT = (M + per_transform<In>() - 1) / per_transform<In>();
    if (c0 >= MT) return;  // a workgroup of the padding (the grid is a multiple of 8)
    const uint32_t cols = MT - c0 < C ? MT - c0 : C;  // transforms
    const uint32_t total = cols * N;
    {
        PackIn<In> v[FFT_EPT];
#pragma unroll
        for (int i = 0; i < FFT_EPT; ++i) {
            const uint32_t e = threadIdx.x + i * DIAG_WG;
            if (e < total) {
                const uint32_t k = e / cols, cl = e - k * cols;
                v[i] = pack_load(src, k, c0 + cl, M);
            }
        }
        for (uint32_t j = threadIdx.x; j < N; j += DIAG_WG) {
            const double2 w = tw[j];
            ftw[j] = make_double2(w.x, sign * w.y);
        }
        const double mid = std::is_same_v<In, uint8_t> ? byte_mid(dst.sums) : 0.0;
#pragma unroll
        for (int i = 0; i < FFT_EPT; ++i) {
            const uint32_t e = threadIdx.x + i * DIAG_WG;
            if (e < total) {
                const uint32_t k = e / cols, cl = e - k * cols;
                fbuf[cl * N + k] = pack_value<In>(v[i], mid);
            }
        }
    }
    __syncthreads();
    uint32_t s = 1;
    for (uint32_t st = 0; st < plan.nst; ++st) {
        const uint32_t R = plan.rad[st];
        if (R == 5) mixed_stage<5>(fbuf, ftw, N, cols, s, sign);
        else if (R == 3) mixed_stage<3>(fbuf, ftw, N, cols, s, sign);
        else if (R == 4) mixed_stage<4>(fbuf, ftw, N, cols, s, sign);
        else mixed_stage<2>(fbuf, ftw, N, cols, s, sign);
        s *= R;
    }
    if constexpr (per_transform<In>() == 1) {
        for (uint32_t e = threadIdx.x; e < total; e += DIAG_WG) {
            const double2 v = fbuf[e];
            const uint32_t cl = e / N;
            pass_store<E>(dst, c0 + cl, e - cl * N, N, M, v.x, v.y);
        }
    } else {
        const uint32_t half = dst.nout;  // N / 2 + 1
        for (uint32_t e = threadIdx.x; e < cols * half; e += DIAG_WG) {
            const uint32_t cl = e / half, k = e - cl * half;
            const double2 *z = fbuf + (size_t)cl * N;
            pair_store<E>(dst, 2 * (c0 + cl), k, N, M, z[k], z[k ? N - k : 0]);
        }
    }
}

// ---- other lengths: Bluestein's chirp convolution ---------------------------------------
//
// With n k = (n^2 + k^2 - (k - n)^2) / 2, the transform X[k] = sum_n x[n] e^{-2 pi i n k / N} is
//   X[k] = c[k] sum_n (x[n] c[n]) b[k - n],   c[n] = e^{-pi i n^2 / N},  b[m] = conj c[m],
// a circular convolution of length M >= 2 N - 1, a power of two, done by two M-point FFTs in one kernel
// (L. Bluestein, 1970).  n^2 mod 2N is exact in integers, so every chirp value is one correctly placed
// sincospi.  The direct pass takes 8 N operations per value, this one about 20 log2 M + 30.
//
// What bounds it is latency: at a side of 1009 the columns are one wave a SIMD, so the FFTs keep their
// values in registers, 16 per thread, and meet in LDS twice each.  M = 16 x 16 x R: with T = M / 16
// threads a column, n = t + T j, t = a + R b and k = k1 + 16 c + 256 d (j, b, c, k1 < 16; a, d < R),
//   forward:  16-point DFTs over j, W_M^{t k1}; over b, W_T^{a c}; R-point DFTs over a;
//   inverse:  the same stages mirrored, so neither needs a reordering pass.
// The forward result lies as X[p + 256 d] at thread p mod T: natural order, in which the transformed
// chirp (the second table, 1/M included) is multiplied in.  The LDS row strides S1 and S2 put the 8 lanes
// of a 128-byte LDS cycle on distinct banks in every exchange.  Real columns go in pairs.
// Against the transform in extended precision the error is below the direct pass's from 80 up: 1.15e-15 of the
// correlation matrix at 1009 x 1009 (direct 3.3e-15), 7.2e-16 at 131 x 137 (1.6e-15), 1.1e-15 at 2039 x
// 2011 (4.5e-15).  Spectrum and correlation matrix, calls back to back: 1009 x 1009 in 40 and 73 us (direct
// 189 and 325), 131 x 137 in 28 and 45 (40 and 72), 2039 x 2011 in 100 and 183 (975 and 1606); a pass at 1009
// takes 14 to 18 us, the tables 8.  83 x 89 in 26 and 42 (30 and 53); at 61 x 67 the direct
// passes take 26 and 42, as long as the convolution at 83.
constexpr uint32_t BLU_MIN = 80, BLU_MAX = 2048;

// Per length N: the chirp c[n] (N entries), the transformed chirp over M (M entries, natural order), then
// the FFTs' twiddles for that M in the order the threads take them: ta[k1 T + t] = W_M^{t k1} and
// tb[16 a + c] = W_T^{a c}.
struct BluTab {
    double2 *c, *b, *ta, *tb;
};
__host__ __device__ constexpr int blu_r(uint32_t N) { return N <= 256 ? 2 : (N <= 512 ? 4 : (N <= 1024 ? 8 : 16)); }
__host__ __device__ constexpr size_t blu_entries(uint32_t N) { return N + (size_t)blu_r(N) * (2 * 256 + 16); }
__host__ __device__ inline BluTab blu_tab(double2 *p, uint32_t N) {
    const size_t m = 256 * (size_t)blu_r(N);
    return BluTab{p, p + N, p + N + m, p + N + 2 * m};
}

__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }

template <int R>
struct BluFft {
    static constexpr int M = 256 * R, T = 16 * R, COLS = DIAG_WG / T;
    static constexpr int S1 = T + (R == 2 ? 2 : (R == 4 ? 4 : 0)), S2 = R == 2 ? 260 : (R == 4 ? 258 : 257);
    static constexpr int COL = 16 * S1 > R * S2 ? 16 * S1 : R * S2;  // LDS entries per column
    static constexpr size_t lds() { return (size_t)COLS * COL * sizeof(double2); }

    static __device__ __forceinline__ void dft_r(double2 *v, double sign) {
        if constexpr (R == 2) {
            const double2 a = v[0];
            v[0] = cadd(a, v[1]);
            v[1] = csub(a, v[1]);
        } else if constexpr (R == 4) {
            dft4(v[0], v[1], v[2], v[3], sign);
        } else if constexpr (R == 8) {
            constexpr double R2 = 0.70710678118654752;  // cos(pi / 4)
            double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
            dft4(e0, e1, e2, e3, sign);
            dft4(o0, o1, o2, o3, sign);
            o1 = cmul(o1, make_double2(R2, sign * R2));
            o2 = rot_q(o2, 1, sign);
            o3 = cmul(o3, make_double2(-R2, sign * R2));
            v[0] = cadd(e0, o0); v[4] = csub(e0, o0);
            v[1] = cadd(e1, o1); v[5] = csub(e1, o1);
            v[2] = cadd(e2, o2); v[6] = csub(e2, o2);
            v[3] = cadd(e3, o3); v[7] = csub(e3, o3);
        } else {
            double2 u[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) u[k] = v[k];
            dft16(u, sign);
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = u[k];
        }
    }

    // v[j] = x[t + T j] -> v[i R + d] = X[i T + t + 256 d].  Each stage's twiddles are loaded before its
    // DFTs; TW gives them (BluTable from memory, or computed).  Every thread of the workgroup calls it, for its barriers;
    // one that is not live leaves L alone.
    template <typename TW>
    static __device__ __forceinline__ void forward(double2 (&v)[16], uint32_t t, double2 *L, const TW &tw,
                                                   double2 (&wa)[16], bool live = true) {
        double2 w[16];
#pragma unroll
        for (int k1 = 1; k1 < 16; ++k1) wa[k1] = tw.a(k1, t);
        dft16(v, -1.0);
        if (live)
#pragma unroll
            for (int k1 = 0; k1 < 16; ++k1) L[k1 * S1 + t] = k1 ? cmul(v[k1], wa[k1]) : v[0];
        const uint32_t k1 = t / R, a = t % R;
#pragma unroll
        for (int c = 1; c < 16; ++c) w[c] = tw.b(a, c);
        __syncthreads();
        if (live)
#pragma unroll
            for (int b = 0; b < 16; ++b) v[b] = L[k1 * S1 + a + R * b];
        __syncthreads();
        dft16(v, -1.0);
        if (live)
#pragma unroll
            for (int c = 0; c < 16; ++c) L[a * S2 + 16 * c + k1] = c ? cmul(v[c], w[c]) : v[0];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16 / R; ++i) {
            if (live)
#pragma unroll
                for (int a2 = 0; a2 < R; ++a2) v[i * R + a2] = L[a2 * S2 + i * T + t];
            dft_r(&v[i * R], -1.0);
        }
    }

    // the way back (without the factor 1/M); starts with a barrier, so that L may still be read before it.  With
    // KEEP, wa still holds the forward transform's first twiddles; otherwise they are loaded again.
    template <bool KEEP, typename TW>
    static __device__ __forceinline__ void inverse(double2 (&v)[16], uint32_t t, double2 *L, const TW &tw,
                                                   double2 (&wa)[16]) {
        const uint32_t k1 = t / R, a = t % R;
        double2 w[16];
#pragma unroll
        for (int c = 1; c < 16; ++c) w[c] = tw.b(a, c);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16 / R; ++i) {
            dft_r(&v[i * R], 1.0);
#pragma unroll
            for (int a2 = 0; a2 < R; ++a2) L[a2 * S2 + i * T + t] = v[i * R + a2];
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            v[c] = L[a * S2 + 16 * c + k1];
            if (c) v[c] = cmul(v[c], conj2(w[c]));
        }
        if constexpr (!KEEP)
#pragma unroll
            for (int k = 1; k < 16; ++k) wa[k] = tw.a(k, t);
        __syncthreads();
        dft16(v, 1.0);
#pragma unroll
        for (int b = 0; b < 16; ++b) L[k1 * S1 + a + R * b] = v[b];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            v[k] = L[k * S1 + t];
            if (k) v[k] = cmul(v[k], conj2(wa[k]));
        }
        dft16(v, 1.0);
    }

    // W_M^{k1 t} and W_T^{a c} (= W_M^{16 a c}), W_M = e^{-2 pi i / M}
    static __device__ __forceinline__ double2 root(uint32_t j) {
        double sn, cs;
        sincospi(2.0 * (double)j / (double)M, &sn, &cs);
        return make_double2(cs, -sn);
    }
    struct FromTable {
        const double2 *ta, *tb;
        __device__ __forceinline__ double2 a(int k1, uint32_t t) const { return ta[k1 * T + t]; }
        __device__ __forceinline__ double2 b(uint32_t a, int c) const { return tb[16 * a + c]; }
    };
    struct Quarter {  // from e^{-2 pi i j / M}, j < M / 4, in LDS (the tables' own workgroup)
        const double2 *q;
        __device__ __forceinline__ double2 at(uint32_t j) const { return rot_q(q[j % (M / 4)], j / (M / 4), -1.0); }
        __device__ __forceinline__ double2 a(int k1, uint32_t t) const { return at(k1 * t); }
        __device__ __forceinline__ double2 b(uint32_t a, int c) const { return at(16 * a * c); }
    };
};

// c[n] = e^{-pi i n^2 / N}
__device__ __forceinline__ double2 chirp(uint32_t n, uint32_t N) {
    const uint32_t e = n * n % (2 * N);  // n < N <= 2048
    double sn, cs;
    sincospi((double)e / (double)N, &sn, &cs);
    return make_double2(cs, -sn);
}

// The tables of length N, by workgroups part = 0 .. parts - 1 (at least 2): the first the chirp and its
// transform (its T first threads hold the column), the others the twiddles.
template <int R>
__device__ __forceinline__ void blu_tables(double2 *p, uint32_t N, uint32_t part, uint32_t parts, double2 *lds) {
    using F = BluFft<R>;
    const BluTab tab = blu_tab(p, N);
    if (part > 0) {
        for (uint32_t i = (part - 1) * DIAG_WG + threadIdx.x; i < F::M + 16 * R; i += (parts - 1) * DIAG_WG) {
            if (i < F::M) tab.ta[i] = F::root((i / F::T) * (i % F::T));
            else tab.tb[i - F::M] = F::root(16 * ((i - F::M) / 16) * (i % 16));
        }
        return;
    }
    double2 *q = lds + F::COL, *cl = q + F::M / 4;
    for (uint32_t j = threadIdx.x; j < F::M / 4; j += DIAG_WG) q[j] = F::root(j);
    for (uint32_t n = threadIdx.x; n < N; n += DIAG_WG) tab.c[n] = cl[n] = chirp(n, N);
    __syncthreads();
    const uint32_t t = threadIdx.x;
    double2 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint32_t n = t + F::T * j, m = n < N ? n : F::M - n;  // b is even
        v[j] = t < F::T && m < N ? conj2(cl[m]) : make_double2(0.0, 0.0);
    }
    // the threads past the column take part in the barriers, all of them outside any branch, and have no place in L
    double2 wa[16];
    F::forward(v, t, lds, typename F::Quarter{q}, wa, t < F::T);
    if (t >= F::T) return;
#pragma unroll
    for (int i = 0; i < 16 / R; ++i)
#pragma unroll
        for (int d = 0; d < R; ++d)
            tab.b[i * F::T + t + 256 * d] = make_double2(v[i * R + d].x * (1.0 / F::M), v[i * R + d].y * (1.0 / F::M));
}

__host__ __device__ constexpr size_t blu_table_lds(uint32_t N) {
    const size_t r = (size_t)blu_r(N), col = r == 2 ? 16 * 34 : (r == 4 ? 16 * 68 : (r == 8 ? 8 * 257 : 16 * 257));
    return (col + 64 * r + N) * sizeof(double2);
}
static_assert(BluFft<2>::COL == 16 * 34 && BluFft<4>::COL == 16 * 68 && BluFft<8>::COL == 8 * 257 && BluFft<16>::COL == 16 * 257,
              "columns of blu_table_lds");

// Workgroups of one launch: a.wgs for the tables of length a.N, b.wgs for those of b.N, and the rest, one
// pair of sums each (Sums).  kind: 0 for the twiddles of the mixed-radix and direct passes, 1 for the chirp
// convolution's tables.
struct TableJob {
    double2 *p;
    uint32_t N, wgs;
    int kind;
};
constexpr uint32_t TABLE_WGS = 9;

__device__ __forceinline__ void make_table(const TableJob &job, uint32_t part, double2 *lds) {
    if (job.kind == 0) {
        for (uint32_t j = part * DIAG_WG + threadIdx.x; j < job.N; j += job.wgs * DIAG_WG) job.p[j] = twiddle_of(j, job.N);
        return;
    }
    switch (blu_r(job.N)) {
        case 2: blu_tables<2>(job.p, job.N, part, job.wgs, lds); break;
        case 4: blu_tables<4>(job.p, job.N, part, job.wgs, lds); break;
        case 8: blu_tables<8>(job.p, job.N, part, job.wgs, lds); break;
        default: blu_tables<16>(job.p, job.N, part, job.wgs, lds); break;
    }
}

// Workgroup `part` of `wgs` of the sums: 16 bytes a load at any alignment, the tail by bytes.
__device__ __forceinline__ void make_sums(const uint8_t *x, uint64_t n, unsigned long long *sums, uint32_t part,
                                          uint32_t wgs) {
    __shared__ unsigned long long red[2][DIAG_WG / 64];
    unsigned long long s1 = 0, s2 = 0;
    auto word = [&](uint32_t w) {
        for (int q = 0; q < 4; ++q) {
            const uint32_t v = (w >> (8 * q)) & 0xFF;
            s1 += v;
            s2 += v * v;
        }
    };
    const uint64_t nv = n / 16;
    for (uint64_t i = (uint64_t)part * DIAG_WG + threadIdx.x; i < nv; i += (uint64_t)wgs * DIAG_WG) {
        uint4 v;
        __builtin_memcpy(&v, x + 16 * i, 16);
        word(v.x);
        word(v.y);
        word(v.z);
        word(v.w);
    }
    if (part == 0 && nv * 16 + threadIdx.x < n) {
        const uint32_t v = x[nv * 16 + threadIdx.x];
        s1 += v;
        s2 += v * v;
    }
    for (int k = 32; k > 0; k >>= 1) {
        s1 += __shfl_xor(s1, k, 64);
        s2 += __shfl_xor(s2, k, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x / 64] = s1;
        red[1][threadIdx.x / 64] = s2;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long t = 0;
        for (int w = 0; w < DIAG_WG / 64; ++w) t += red[threadIdx.x][w];
        sums[2 * part + threadIdx.x] = t;
    }
}

__global__ __launch_bounds__(DIAG_WG) void tables_kernel(TableJob a, TableJob b, const uint8_t *img, uint64_t n,
                                                         unsigned long long *sums) {
    extern __shared__ double2 fbuf[];
    uint32_t part = blockIdx.x;
    if (part < a.wgs) return make_table(a, part, fbuf);
    part -= a.wgs;
    if (part < b.wgs) return make_table(b, part, fbuf);
    part -= b.wgs;
    make_sums(img, n, sums, part, gridDim.x - a.wgs - b.wgs);
}

// KEEP: the first stage's twiddles stay in registers between the two FFTs, at more than 256 of them, so one
// workgroup a CU.
template <typename In, int E, int R, bool KEEP>
__global__ __launch_bounds__(DIAG_WG) void blu_pass_kernel(const In *src, uint32_t N, uint32_t M, const BluTab tab,
                                                            double sign, PassOut dst) {
    using F = BluFft<R>;
    pass_sums<E>(dst);
    extern __shared__ double2 fbuf[];
    constexpr bool REAL = !std::is_same_v<In, double2>;
    const uint32_t t = threadIdx.x % F::T, sub = threadIdx.x / F::T;
    double2 *L = fbuf + (size_t)sub * F::COL;
    const typename F::FromTable tw{tab.ta, tab.tb};
    // consecutive column groups on the same XCD (the grid is a multiple of 8)
    const uint32_t g = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    const uint32_t tr = g * F::COLS + sub, col = tr * per_transform<In>();
    const bool one = col < M;
    // N <= M / 2: rows t + T j, j < 8.  All loads first: the column's and the chirp's.
    PackIn<In> x[8];
    double2 ch[8], v[16];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t n = t + F::T * j;
        x[j] = PackIn<In>{};
        ch[j] = make_double2(0.0, 0.0);
        if (one && n < N) x[j] = pack_load(src, n, tr, M);
        if (n < N) ch[j] = tab.c[n];
    }
    const double mid = std::is_same_v<In, uint8_t> ? byte_mid(dst.sums) : 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        double2 z = pack_value<In>(x[j], mid);
        if (sign > 0) z.y = -z.y;  // the transform of the other sign: conjugated in and out
        v[j] = cmul(z, ch[j]);     // zero past the last row, with its chirp
        v[j + 8] = make_double2(0.0, 0.0);
    }
    double2 wa[16];
    F::forward(v, t, L, tw, wa);
#pragma unroll
    for (int i = 0; i < 16 / R; ++i)
#pragma unroll
        for (int d = 0; d < R; ++d) v[i * R + d] = cmul(v[i * R + d], tab.b[i * F::T + t + 256 * d]);
    F::template inverse<KEEP>(v, t, L, tw, wa);
    if constexpr (!REAL) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t n = t + F::T * j;
            if (one && n < N) {
                const double2 z = cmul(v[j], ch[j]);
                pass_store<E>(dst, col, n, N, M, z.x, sign > 0 ? -z.y : z.y);
            }
        }
    } else {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t n = t + F::T * j;
            if (n < N) {
                const double2 z = cmul(v[j], ch[j]);
                L[n] = make_double2(z.x, sign > 0 ? -z.y : z.y);
            }
        }
        __syncthreads();
        if (!one) return;
        for (uint32_t k = t; k < dst.nout; k += F::T) {
            pair_store<E>(dst, col, k, N, M, L[k], L[k ? N - k : 0]);
        }
    }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int check_matrix(const lz_ctx *c, const uint8_t *img, uint32_t h, uint32_t w, const void *out) {
    if (!c || !img || !out) return fail(LZ_E_INVAL, "NULL argument");
    if (h == 0 || w == 0) return fail(LZ_E_INVAL, "empty matrix");
    if (h > 65536 || w > 65536 || (uint64_t)h * w > (1ull << 24))
        return fail(LZ_E_INVAL, "matrix too large: h, w <= 65536 and h * w <= 2^24");
    return LZ_OK;
}

struct Dft2 {
    unsigned long long *sums;
    double2 *tw_h, *tw_w, *a, *b;
};

// Entries of length N's table: its twiddles, or the chirp and its transform.
size_t table_entries(uint32_t N) { return N <= BLU_MAX ? blu_entries(N) : N; }

constexpr size_t SUMS_BYTES = (size_t)SUM_WGS * 2 * sizeof(unsigned long long);

// Workspace: the sums, tables for h and w, then two h*w complex buffers.
Dft2 dft2_layout(char *ws, uint32_t h, uint32_t w) {
    Dft2 d;
    size_t off = align256(SUMS_BYTES);
    d.sums = reinterpret_cast<unsigned long long *>(ws);
    d.tw_h = reinterpret_cast<double2 *>(ws + off);
    off += align256(table_entries(h) * sizeof(double2));
    d.tw_w = reinterpret_cast<double2 *>(ws + off);
    off += align256(table_entries(w) * sizeof(double2));
    d.a = reinterpret_cast<double2 *>(ws + off);
    off += align256((size_t)h * w * sizeof(double2));
    d.b = reinterpret_cast<double2 *>(ws + off);
    return d;
}

size_t dft2_bytes(uint32_t h, uint32_t w) {
    return align256(SUMS_BYTES) + align256(table_entries(h) * sizeof(double2)) +
           align256(table_entries(w) * sizeof(double2)) + 2 * align256((size_t)h * w * sizeof(double2));
}

// The radices of N for the mixed-radix pass (5s, 3s, 4s, then a 2), or nst = 0 if N has
// another prime factor.
FftPlan mixed_plan(uint32_t N) {
    FftPlan p{};
    uint32_t n = N;
    for (uint32_t r : {5u, 3u}) {
        while (n % r == 0 && p.nst < 16) {
            p.rad[p.nst++] = (uint8_t)r;
            n /= r;
        }
    }
    while (n % 4 == 0 && p.nst < 16) {
        p.rad[p.nst++] = 4;
        n /= 4;
    }
    if (n == 2 && p.nst < 16) {
        p.rad[p.nst++] = 2;
        n = 1;
    }
    if (n != 1) p.nst = 0;
    return p;
}

size_t mixed_lds(uint32_t N) {
    const uint32_t per_wg = N > FFT_WG_ELEMS ? N : FFT_WG_ELEMS;
    return ((size_t)(per_wg / N) * N + N) * sizeof(double2);
}

bool mixed_ok(const lz_ctx *c, uint32_t N) {
    return N <= FFT_MAX && N > 1 && mixed_plan(N).nst > 0 && mixed_lds(N) <= (size_t)c->dev.lds_per_wg_max;
}

size_t fft_lds(uint32_t N) {
    const uint32_t per_wg = N > FFT_WG_ELEMS ? N : FFT_WG_ELEMS;
    return ((size_t)(N <= FFT_PP_MAX ? 2 : 1) * per_wg + fft_twiddles(N)) * sizeof(double2);
}

bool fft_ok(const lz_ctx *c, uint32_t N) {
    const size_t lds = fft_lds(N);
    return (N & (N - 1)) == 0 && N <= FFT_MAX && lds <= (size_t)c->dev.lds_per_wg_max;
}

size_t blu_lds(uint32_t N) {
    switch (blu_r(N)) {
        case 2: return BluFft<2>::lds();
        case 4: return BluFft<4>::lds();
        case 8: return BluFft<8>::lds();
        default: return BluFft<16>::lds();
    }
}

// Lengths for the chirp convolution: those with a prime factor above 5 from BLU_MIN on, where it takes over from
// the direct pass in time and error, up to BLU_MAX, whose convolution of 4096 points a workgroup's LDS holds.
bool blu_ok(const lz_ctx *c, uint32_t N) {
    return N >= BLU_MIN && N <= BLU_MAX && !fft_ok(c, N) && !mixed_ok(c, N) &&
           blu_lds(N) <= (size_t)c->dev.lds_per_wg_max && blu_table_lds(N) <= (size_t)c->dev.lds_per_wg_max;
}

// One launch for the tables of the lengths that are not powers of two (the power-of-two FFT makes its own;
// equal sides share one) and the sums over the bytes, if anything needs them: the correlation matrix does,
// and a spectrum with a table to make takes the mean out as well.
int launch_tables(const lz_ctx *c, Dft2 &d, const uint8_t *img, uint32_t h, uint32_t w, bool need_sums, Sums *sums,
                  hipStream_t s) {
    if (h == w) d.tw_w = d.tw_h;
    TableJob a{}, b{};
    size_t lds = 0;
    auto job = [&](double2 *p, uint32_t N) {
        TableJob t{p, N, 0, blu_ok(c, N) ? 1 : 0};
        if (fft_ok(c, N)) return t;
        t.wgs = t.kind ? TABLE_WGS : (N + DIAG_WG - 1) / DIAG_WG;
        if (t.kind && blu_table_lds(N) > lds) lds = blu_table_lds(N);
        return t;
    };
    a = job(d.tw_h, h);
    if (h != w) b = job(d.tw_w, w);
    *sums = Sums{nullptr, 0, (uint64_t)h * w};
    if (!need_sums && !a.wgs && !b.wgs) return LZ_OK;
    const uint64_t want = (sums->n + 16383) / 16384;  // 16 KiB a workgroup at least
    sums->wgs = want < SUM_WGS ? (uint32_t)want : SUM_WGS;
    sums->p = d.sums;
    if (lds > 65536)
        LZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&tables_kernel),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(tables_kernel, dim3(a.wgs + b.wgs + sums->wgs), dim3(DIAG_WG), lds, s, a, b, img, sums->n, d.sums);
    LZ_HIP(hipGetLastError());
    return LZ_OK;
}

// The twiddles stay in registers (KEEP) where the grid leaves room for one workgroup a CU at most: 2 and 4 us of
// 1009 x 1009's; at 2039 x 2011, four workgroups a CU, it would be 133 and 252 us instead of 106 and 203 (the same run).
template <typename In, int E, int R>
int launch_blu(const lz_ctx *c, const In *src, uint32_t N, uint32_t M, const double2 *table, double sign, PassOut out,
               hipStream_t s) {
    using F = BluFft<R>;
    const uint32_t cols = std::is_same_v<In, double2> ? M : (M + 1) / 2;
    const uint32_t groups = ((cols + F::COLS - 1) / F::COLS + 7) / 8 * 8;  // a multiple of 8: the XCD-aware order
    const BluTab tab = blu_tab(const_cast<double2 *>(table), N);
    auto run = [&](auto keep) -> int {
        constexpr bool KEEP = decltype(keep)::value;
        if (F::lds() > 65536)
            LZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&blu_pass_kernel<In, E, R, KEEP>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)F::lds()));
        hipLaunchKernelGGL((blu_pass_kernel<In, E, R, KEEP>), dim3(groups), dim3(DIAG_WG), F::lds(), s, src, N, M, tab,
                           sign, out);
        return LZ_OK;
    };
    if (int rc = groups <= (uint32_t)c->dev.cus ? run(std::true_type{}) : run(std::false_type{})) return rc;
    LZ_HIP(hipGetLastError());
    return LZ_OK;
}

// Output (M x out.nout) = transpose of (DFT_N along the rows of src (N x M)), its first out.nout
// rows, stored by epilogue E: by FFT when N is a power of two up to FFT_MAX, by mixed-radix FFT
// when N <= FFT_MAX has no prime factor above 5, by chirp convolution where blu_ok, otherwise directly
// on the matrix cores (tw: the length's table, needed by the last three).
template <typename In, int E>
int launch_dft_pass(const lz_ctx *c, const In *src, uint32_t N, uint32_t M, const double2 *tw, double sign,
                    PassOut out, hipStream_t s) {
    if (N == FFT1K && fft1k_lds() <= (size_t)c->dev.lds_per_wg_max) {
        const size_t lds = fft1k_lds();
        if (lds > 65536)
            LZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&fft1k_pass_kernel<In, E>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        // a multiple of 8 workgroups, so that neighbouring column groups share an XCD (the
        // workgroups past the last column only help make the twiddle table and leave)
        const uint32_t groups = ((M + FFT1K_COLS - 1) / FFT1K_COLS + 7) / 8 * 8;
        hipLaunchKernelGGL((fft1k_pass_kernel<In, E>), dim3(groups), dim3(DIAG_WG), lds, s, src, M, sign, out);
    } else if (fft_ok(c, N)) {
        uint32_t logN = 0;
        while ((1u << logN) < N) ++logN;
        const uint32_t per_wg = N > FFT_WG_ELEMS ? N : FFT_WG_ELEMS;
        const uint32_t C = per_wg / N;
        const uint32_t groups = ((M + C - 1) / C + 7) / 8 * 8;  // a multiple of 8: the XCD-aware order
        const size_t lds = fft_lds(N);
        if (lds > 65536)
            LZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&fft_pass_kernel<In, E>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL((fft_pass_kernel<In, E>), dim3(groups), dim3(DIAG_WG), lds, s, src, N, M, logN, C, sign,
                           out);
    } else if (mixed_ok(c, N)) {
        const uint32_t per_wg = N > FFT_WG_ELEMS ? N : FFT_WG_ELEMS;
        const uint32_t C = per_wg / N;
        const uint32_t MT = (M + per_transform<In>() - 1) / per_transform<In>();
        const uint32_t groups = ((MT + C - 1) / C + 7) / 8 * 8;  // a multiple of 8: the XCD-aware order
        const size_t lds = mixed_lds(N);
        if (lds > 65536)
            LZ_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&fft_mixed_pass_kernel<In, E>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL((fft_mixed_pass_kernel<In, E>), dim3(groups), dim3(DIAG_WG), lds, s, src, N, M, C,
                           mixed_plan(N), tw, sign, out);
    } else if (blu_ok(c, N)) {
        switch (blu_r(N)) {
            case 2: return launch_blu<In, E, 2>(c, src, N, M, tw, sign, out, s);
            case 4: return launch_blu<In, E, 4>(c, src, N, M, tw, sign, out, s);
            case 8: return launch_blu<In, E, 8>(c, src, N, M, tw, sign, out, s);
            default: return launch_blu<In, E, 16>(c, src, N, M, tw, sign, out, s);
        }
    } else {
        // 64 x 64 tiles, or 32 x 64 where those would leave compute units idle; DFT_KS32 and
        // DFT_KS64 terms per LDS stage (the smaller tiles do half the products per term)
        const uint32_t gy = (M + DFT_T - 1) / DFT_T;
        if ((uint64_t)((out.nout + DFT_T - 1) / DFT_T) * gy < (uint64_t)c->dev.cus) {
            const dim3 grid((out.nout + 31) / 32, gy);
            hipLaunchKernelGGL((dft_pass_kernel<In, E, 32, DFT_KS32>), grid, dim3(DIAG_WG), 0, s, src, N, M, tw,
                               sign, out);
        } else {
            const dim3 grid((out.nout + DFT_T - 1) / DFT_T, gy);
            hipLaunchKernelGGL((dft_pass_kernel<In, E, 64, DFT_KS64>), grid, dim3(DIAG_WG), 0, s, src, N, M, tw,
                               sign, out);
        }
    }
    LZ_HIP(hipGetLastError());
    return LZ_OK;
}

// complex results, indices r < nout of each transform; real results, whole rows of n, with the
// mirror rows of an h-row matrix (0: none).  sums: for a pass over bytes and for the last pass.
PassOut complex_out(double2 *z, uint32_t nout, const Sums &sums = Sums{}) {
    return PassOut{z, nullptr, nout, 0, sums, 0.0, 0.0};
}
PassOut real_out(double *p, uint32_t n, uint32_t h, const Sums &sums = Sums{}) {
    return PassOut{nullptr, p, n, h, sums, 0.0, 0.0};
}

}  // namespace
}  // namespace lz

using namespace lz;

extern "C" int lz_power_spectrum_2d(lz_ctx *c, const uint8_t *d_img, uint32_t h, uint32_t w, double *d_power,
                                    void *stream) {
    if (int rc = check_matrix(c, d_img, h, w, d_power)) return rc;
    hipStream_t s = (hipStream_t)stream;
    LZ_HIP(hipSetDevice(c->device));
    char *ws;
    if (int rc = diag_begin(c, s, dft2_bytes(h, w), &ws)) return rc;
    Dft2 d = dft2_layout(ws, h, w);
    Sums sums;
    if (int rc = launch_tables(c, d, d_img, h, w, false, &sums, s)) return rc;
    // a: w x (h/2 + 1), the columns' transforms up to index h/2 (the rest is their mirror image);
    // then |Z|^2 of the second pass, rows 0..h/2 and their mirror rows, straight into the output
    const uint32_t hh = h / 2 + 1;
    if (int rc = launch_dft_pass<uint8_t, EPI_COMPLEX>(c, d_img, h, w, d.tw_h, -1.0, complex_out(d.a, hh, sums), s))
        return rc;
    if (int rc = launch_dft_pass<double2, EPI_POWER>(c, d.a, w, hh, d.tw_w, -1.0, real_out(d_power, w, h, sums), s))
        return rc;
    return diag_end(c, s);
}

extern "C" int lz_autocorrelation_2d(lz_ctx *c, const uint8_t *d_img, uint32_t h, uint32_t w, double *d_acf,
                                     void *stream) {
    if (int rc = check_matrix(c, d_img, h, w, d_acf)) return rc;
    hipStream_t s = (hipStream_t)stream;
    LZ_HIP(hipSetDevice(c->device));
    char *ws;
    if (int rc = diag_begin(c, s, dft2_bytes(h, w), &ws)) return rc;
    Dft2 d = dft2_layout(ws, h, w);
    Sums sums;
    if (int rc = launch_tables(c, d, d_img, h, w, true, &sums, s)) return rc;
    // a: w x (h/2 + 1); b: |Z|^2 with the zero frequency removed (h x w, real and even); a: w x (h/2 + 1)
    // again; then Re G / den, den = n S2 - S1^2 from the sums, rows 0..h/2 and their mirror rows (G is
    // even too)
    const uint32_t hh = h / 2 + 1;
    double *pm = reinterpret_cast<double *>(d.b);
    if (int rc = launch_dft_pass<uint8_t, EPI_COMPLEX>(c, d_img, h, w, d.tw_h, -1.0, complex_out(d.a, hh, sums), s))
        return rc;
    if (int rc = launch_dft_pass<double2, EPI_POWER_NODC>(c, d.a, w, hh, d.tw_w, -1.0, real_out(pm, w, h), s))
        return rc;
    if (int rc = launch_dft_pass<double, EPI_COMPLEX>(c, pm, h, w, d.tw_h, 1.0, complex_out(d.a, hh), s))
        return rc;
    if (int rc = launch_dft_pass<double2, EPI_ACF>(c, d.a, w, hh, d.tw_w, 1.0, real_out(d_acf, w, h, sums), s))
        return rc;
    return diag_end(c, s);
}
