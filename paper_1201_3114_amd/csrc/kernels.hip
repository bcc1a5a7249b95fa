// gfx950 kernels of the Lorenz chaotic cipher (arXiv:1201.3114, Sections 3
// and 5).  One lane carries M independent chains (blocks of the parallel
// version); the per-byte work is Steps 1-3 of Section 3.2, dominated by
// n_it forward-Euler steps of the Lorenz system in binary64 (14 roundings per
// step, no contraction: the file is built with -ffp-contract=off and nothing
// here may be fused, so results equal the exact IEEE sequence of the method).
//
// Byte streams: a wave stages `tile` bytes of each of its 64*M chains into
// LDS with lane-contiguous (coalesced) global loads, the lanes consume their
// own chain's bytes from LDS, write the output bytes back in place, and the
// wave stores the tile with lane-contiguous global stores.
//
// A call with fewer chains than the chip has lanes takes its chains' serial
// time, which is the number of instructions of one step times four clocks.  For
// these a chain spreads over the 4 lanes of a quad or the 16 of a row, one
// coordinate per lane or bank (G = 4, 16 below): the three coordinates'
// operations share instructions.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "internal.h"

namespace lz {
namespace {

constexpr double SIGMA = 10.0;
constexpr double RHO = 28.0;
constexpr double BETA = 8.0 / 3.0;
constexpr double SCALE_NU = 1e13;  // 10^nu, nu = floor(log10 2^(52-6)) = 13
constexpr int WAVE = 64;

// ---- scalar pieces of the method ------------------------------------------------

__device__ __forceinline__ double sel3(uint32_t m, double x, double y, double z) {
    return m == 0 ? x : (m == 1 ? y : z);
}

// Eq. R_nu: byte Omega (0..3) of floor(alpha 10^13) in two's complement.  The
// integer N has |N| < 2^53; N mod 2^32 is formed exactly in binary64.
__device__ __forceinline__ uint32_t r_nu(double alpha, uint32_t om) {
    const double N = floor(alpha * SCALE_NU);
    const double hi = floor(N * 0x1p-32);
    const double lo = N - hi * 0x1p32;
    return ((uint32_t)lo >> (8u * om)) & 0xFFu;
}

// Step 2: Theta = P / 10^(3 + Omega_3), one correctly rounded division.
__device__ __forceinline__ double theta_of(uint32_t p, uint32_t o3) {
    const double p10 = o3 == 0 ? 1e3 : (o3 == 1 ? 1e4 : (o3 == 2 ? 1e5 : 1e6));
    return (double)p / p10;
}

// Integrity word N(v) = floor(v 10^13) as a two's complement 64-bit pattern.
__device__ __forceinline__ unsigned long long digest_word(double v) {
    const double N = floor(v * SCALE_NU);
    const double hi = floor(N * 0x1p-32);
    const double lo = N - hi * 0x1p32;
    return ((unsigned long long)(uint32_t)(int32_t)hi << 32) | (unsigned long long)(uint32_t)lo;
}

// Section 3.1: one forward Euler step of the Lorenz system, fixed order.
__device__ __forceinline__ void euler_step(double &x, double &y, double &z, double dt) {
    const double dx = SIGMA * (y - x);
    const double dy = (x * (RHO - z)) - y;
    const double dz = (x * y) - (BETA * z);
    x = x + dt * dx;
    y = y + dt * dy;
    z = z + dt * dz;
}

// Format variant: the Euler step with each update fused into one rounding (9 roundings).
__device__ __forceinline__ void euler_fma_step(double &x, double &y, double &z, double dt) {
    const double dx = SIGMA * (y - x);
    const double dy = __builtin_fma(x, RHO - z, -y);
    const double dz = __builtin_fma(x, y, -(BETA * z));
    x = __builtin_fma(dt, dx, x);
    y = __builtin_fma(dt, dy, y);
    z = __builtin_fma(dt, dz, z);
}

// Lorenz vector field in the Euler step's evaluation order.
__device__ __forceinline__ void lorenz_field(double x, double y, double z, double &fx, double &fy, double &fz) {
    fx = SIGMA * (y - x);
    fy = (x * (RHO - z)) - y;
    fz = (x * y) - (BETA * z);
}

// v + 2 u: 2 u is exact, so the one rounding of the fused form is that of the sum.  In assembly because the
// compiler's choice, v_fmac_f64, is a 4-byte instruction, which moves the 8-byte ones after it in
// the step loop off their fetch words.
__device__ __forceinline__ double twice_plus(double u, double v) {
    double r;
    asm("v_fma_f64 %0, %1, 2.0, %2" : "=v"(r) : "v"(u), "v"(v));
    return r;
}

// Format variant: classical Runge-Kutta 4, r += dt/6 ((k1 + k4) + 2 (k2 + k3)).
__device__ __forceinline__ void rk4_step(double &x, double &y, double &z, double dt, double h2, double h6) {
    double ax, ay, az, bx, by, bz, cx, cy, cz, dx, dy, dz;
    lorenz_field(x, y, z, ax, ay, az);
    lorenz_field(x + h2 * ax, y + h2 * ay, z + h2 * az, bx, by, bz);
    lorenz_field(x + h2 * bx, y + h2 * by, z + h2 * bz, cx, cy, cz);
    lorenz_field(x + dt * cx, y + dt * cy, z + dt * cz, dx, dy, dz);
    x = x + h6 * twice_plus(bx + cx, ax + dx);
    y = y + h6 * twice_plus(by + cy, ay + dy);
    z = z + h6 * twice_plus(bz + cz, az + dz);
}

template <int I>
__device__ __forceinline__ void step(double &x, double &y, double &z, double dt, double h2, double h6) {
    if constexpr (I == LZ_INTEGRATOR_EULER_FMA) euler_fma_step(x, y, z, dt);
    else if constexpr (I == LZ_INTEGRATOR_RK4) rk4_step(x, y, z, dt, h2, h6);
    else euler_step(x, y, z, dt);
}

// A counted loop of STEP (N instructions, 8 bytes each), U steps an iteration and %[q] + 1 iterations, none if %[q]
// is -1.  The first iteration is entered %[at] bytes on, where the steps are left to run that U does not divide.  A wave
// alone on its SIMD pays four clocks for each scalar instruction too: U = 120 (8 to 13 KB of code) and two scalar
// instructions an iteration, instead of 60 and three, are 0.3% at four waves per SIMD; 20 steps an iteration
// cost 2%.  With the entry every step count costs its steps: 16 MiB at 100 steps a byte take 0.91 ms (fused map
// 0.70), 1.25 (1.03) with the remainder in a loop of single steps, 0.94 (0.73) in one of twelve. Where none is left
// over a branch goes to the loop: by address 3 MB took 14.59 ms, 14.51 by the branch.
#define LZ_STEP_LOOP(U, N, STEP)                                               \
    "s_nop 4\n"                                                                \
    "s_cmp_lt_i32 %[q], 0\n"                                                   \
    "s_cbranch_scc1 4f\n"                                                      \
    "s_cmp_eq_u32 %[at], 0\n"                                                  \
    "s_cbranch_scc1 2f\n"                                                      \
    "s_getpc_b64 s[40:41]\n"                                                   \
    "1:\n"                                                                     \
    "s_add_u32 s40, s40, %[at]\n"                                              \
    "s_addc_u32 s41, s41, 0\n"                                                 \
    "s_add_u32 s40, s40, 2f-1b\n"                                              \
    "s_addc_u32 s41, s41, 0\n"                                                 \
    "s_setpc_b64 s[40:41]\n"                                                   \
    ".p2align 6\n"                                                             \
    "2:\n"                                                                     \
    ".rept " #U "\n" STEP ".endr\n"                                            \
    "3:\n"                                                                     \
    ".if (3b - 2b) != " #U " * " #N " * 8\n"                                   \
    ".error \"a step of another length\"\n"                                    \
    ".endif\n"                                                                 \
    "s_sub_u32 %[q], %[q], 1\n"                                                \
    "s_cbranch_scc0 2b\n"                                                      \
    "4:\n"                                                                     \
    "s_nop 1\n"
#define LZ_STEP_CLOBBER "scc", "s40", "s41"
constexpr uint32_t STEP_U = 120, RK4_U = 60;  // RK4: 22 KB, a step is 43 or 47 instructions

// The operands for n_it steps of n instructions, u an iteration.
struct StepCount {
    uint32_t q, at;
    __device__ StepCount(uint32_t n_it, uint32_t u, uint32_t n)
        : q(n_it / u + (n_it % u != 0) - 1), at(n_it % u ? (u - n_it % u) * n * 8 : 0) {}
};

// F^(n_it) of one chain per lane, for the two Euler maps: the instructions of euler_step and euler_fma_step in
// an order of our own.  With all SIMDs busy the part's power decides the clock, and the order of a step's
// instructions decides the power: like operations next to each other, the three products with dt in a row, draw
// less than the compiler's interleaving.  Of 160 random valid orders of the 14 instructions (24 ms launches of
// four waves per SIMD, three times each) the times ran from 36.97 to 38.08 ms per 384000 steps; the
// compiler's order took 37.83, this one 37.00 (35.84 at 2.4 GHz).  64 MiB, the two orders in turn on three cards: 77.0 to 78.1 ms
// in the compiler's and 74.7 to 75.1 in this one, 76.0 to 76.7 and 74.0 to 74.2, 74.3 to 74.6 and 73.7 to 73.8.  For the
// fused map 80 orders ran from 37.85 (this one) to 39.69, and the compiler's is one of the fast ones: 51.3 to 52.0 ms
// for 64 MiB, 51.4 to 52.2 in this one.
template <int I>
__device__ __forceinline__ void lane_steps(double &x, double &y, double &z, double dt, uint32_t n_it) {
    double d, e, f, g;
    StepCount n(n_it, STEP_U, I == LZ_INTEGRATOR_EULER_FMA ? 9 : 14);
    if constexpr (I == LZ_INTEGRATOR_EULER_FMA) {
        asm volatile(LZ_STEP_LOOP(120, 9,
                         "v_add_f64 %[e], -%[z], %[rho]\n"
                         "v_add_f64 %[d], %[y], -%[x]\n"
                         "v_mul_f64 %[d], %[d], %[sigma]\n"
                         "v_mul_f64 %[g], %[z], %[beta]\n"
                         "v_fma_f64 %[e], %[x], %[e], -%[y]\n"
                         "v_fma_f64 %[f], %[x], %[y], -%[g]\n"
                         "v_fma_f64 %[x], %[dt], %[d], %[x]\n"
                         "v_fma_f64 %[y], %[dt], %[e], %[y]\n"
                         "v_fma_f64 %[z], %[dt], %[f], %[z]\n")
                     : [x] "+v"(x), [y] "+v"(y), [z] "+v"(z), [d] "=&v"(d), [e] "=&v"(e), [f] "=&v"(f), [g] "=&v"(g),
                       [q] "+s"(n.q)
                     : [at] "s"(n.at), [dt] "s"(dt), [sigma] "s"(SIGMA), [rho] "s"(RHO), [beta] "s"(BETA)
                     : LZ_STEP_CLOBBER);
    } else {
        static_assert(I == LZ_INTEGRATOR_EULER, "the two Euler maps");
        asm volatile(LZ_STEP_LOOP(120, 14,
                         "v_add_f64 %[e], -%[z], %[rho]\n"
                         "v_add_f64 %[d], %[y], -%[x]\n"
                         "v_mul_f64 %[f], %[x], %[y]\n"
                         "v_mul_f64 %[e], %[x], %[e]\n"
                         "v_mul_f64 %[g], %[z], %[beta]\n"
                         "v_mul_f64 %[d], %[d], %[sigma]\n"
                         "v_add_f64 %[e], %[e], -%[y]\n"
                         "v_add_f64 %[f], %[f], -%[g]\n"
                         "v_mul_f64 %[d], %[dt], %[d]\n"
                         "v_mul_f64 %[e], %[dt], %[e]\n"
                         "v_mul_f64 %[f], %[dt], %[f]\n"
                         "v_add_f64 %[x], %[x], %[d]\n"
                         "v_add_f64 %[y], %[y], %[e]\n"
                         "v_add_f64 %[z], %[z], %[f]\n")
                     : [x] "+v"(x), [y] "+v"(y), [z] "+v"(z), [d] "=&v"(d), [e] "=&v"(e), [f] "=&v"(f), [g] "=&v"(g),
                       [q] "+s"(n.q)
                     : [at] "s"(n.at), [dt] "s"(dt), [sigma] "s"(SIGMA), [rho] "s"(RHO), [beta] "s"(BETA)
                     : LZ_STEP_CLOBBER);
    }
}

// Step 2's F^(n_it) for the M chains of a lane, interleaved step by step.
template <int M, int I>
__device__ __forceinline__ void lorenz_steps(double (&x)[M], double (&y)[M], double (&z)[M], double dt,
                                             uint32_t n_it) {
    if constexpr (M == 1 && I != LZ_INTEGRATOR_RK4) return lane_steps<I>(x[0], y[0], z[0], dt, n_it);
    const double h2 = dt * 0.5, h6 = I == LZ_INTEGRATOR_RK4 ? dt / 6.0 : 0.0;
    // Steps per loop iteration: 60 / M Euler steps for M chains (a divisor of the default 3000, about 6.7 KB
    // of code); RK4's 65-operation step gains nothing from more.
    constexpr int U = I == LZ_INTEGRATOR_RK4 ? 2 : 60 / M;
    const uint32_t q = n_it / U;
    for (uint32_t i = 0; i < q; ++i) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int m = 0; m < M; ++m) step<I>(x[m], y[m], z[m], dt, h2, h6);
        }
    }
    for (uint32_t i = q * U; i < n_it; ++i) {
#pragma unroll
        for (int m = 0; m < M; ++m) step<I>(x[m], y[m], z[m], dt, h2, h6);
    }
}

// ---- one chain over the lanes of a quad -----------------------------------------------
//
// With one wave on a SIMD a vector instruction takes four clocks, dependent or not, so a step costs
// its instruction count: 14 with a chain per lane.  In a quad, lane 0 holds x, lane 1 y, lane 2 z
// and lane 3 the constant sigma; with per-lane constants (m, c, k, s) every lane computes
//
//     q = m v + c            (-x, rho, 0)       t = s P1 + q    (y - x, rho - z, y)
//     u = k v                (0, y, beta z)     t = t P2        (sigma (y-x), x (rho-z), x y)
//     P1 = v of lanes 1,2,1                     t = t - u       (dx, dy, dz)
//     P2 = v of lanes 3,0,0                     v = v + dt t
//
// 7 binary64 instructions and 4 32-bit moves between lanes, 11 in all.  Each lane's value goes through the same
// roundings as in euler_step: the factors m, s and k are 0, 1 or -1 except k = beta, so the products
// they form are exact (a zero's sign may differ, its value not).  Measured with one wave per SIMD:
// 44.6 clocks per step against 56.6 with a chain per lane.  A wave holds 16 chains instead of 64.
//
// The loops are written in assembly for two reasons: a lane's value must stay in a register pair
// whose halves the moves can name, and every instruction in them is 8 bytes long.  One 4-byte
// instruction shifts all that follow across the 8-byte fetch words, which costs 25% (70.5 clocks per
// step instead of 56.6 for the one-lane loop).  Two instructions lie between the write of v and the
// first move that reads it through DPP, which must not follow within two wait states.

template <int G>
struct LaneRole {};

template <>
struct LaneRole<4> {
    double m, c, k, s;
    __device__ explicit LaneRole(int lane) {
        const int r = lane & 3;
        m = r == 0 ? -1.0 : 0.0;
        c = r == 1 ? RHO : 0.0;
        k = r == 1 ? 1.0 : (r == 2 ? BETA : 0.0);
        s = r == 3 ? 0.0 : (r == 1 ? -1.0 : 1.0);
    }
};
template <>
struct LaneRole<16> {
    double m, k, s, one;
    __device__ explicit LaneRole(int lane) {
        const int r = (lane >> 2) & 3;
        m = r == 0 ? -1.0 : 0.0;
        k = r == 1 ? 1.0 : (r == 2 ? BETA : 0.0);
        s = r == 3 ? 0.0 : (r == 1 ? -1.0 : 1.0);
        one = 1.0;
    }
};
template <>
struct LaneRole<1> {
    __device__ explicit LaneRole(int) {}
};

// The value of `v` in the lane that DPP control CTRL names.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)((unsigned long long)b >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The vector field of the value in v[LO:HI] into OUT (P1 in v[60:61], P2 in v[62:63]).
#define LZ_QUAD_FIELD(LO, HI, OUT)                                                             \
    "v_fma_f64 %[q0], %[m], v[" LO ":" HI "], %[c]\n"                                          \
    "v_mul_f64 %[u], %[k], v[" LO ":" HI "]\n"                                                 \
    "v_mov_b32_dpp v60, v" LO " quad_perm:[1,2,1,3] row_mask:0xf bank_mask:0xf\n"              \
    "v_mov_b32_dpp v61, v" HI " quad_perm:[1,2,1,3] row_mask:0xf bank_mask:0xf\n"              \
    "v_mov_b32_dpp v62, v" LO " quad_perm:[3,0,0,3] row_mask:0xf bank_mask:0xf\n"              \
    "v_mov_b32_dpp v63, v" HI " quad_perm:[3,0,0,3] row_mask:0xf bank_mask:0xf\n"              \
    "v_fma_f64 " OUT ", %[s], v[60:61], %[q0]\n"                                               \
    "v_mul_f64 " OUT ", " OUT ", v[62:63]\n"                                                   \
    "v_add_f64 " OUT ", " OUT ", -%[u]\n"

// n_it steps of the chain whose coordinates x, y, z all lanes of the quad hold.
template <int I>
__device__ __forceinline__ void quad_steps(double &x, double &y, double &z, double dt, uint32_t n_it,
                                           const LaneRole<4> &role, int lane) {
    const int lr = lane & 3;
    double v = lr == 0 ? x : (lr == 1 ? y : (lr == 2 ? z : SIGMA));
    constexpr uint32_t U = I == LZ_INTEGRATOR_RK4 ? RK4_U : STEP_U;
    StepCount n(n_it, U, I == LZ_INTEGRATOR_RK4 ? 47 : 11);
    double q0, u, t, p1, p2;
    if constexpr (I == LZ_INTEGRATOR_RK4) {
        // the field four times (9 instructions each) and the 11 operations of rk4_step between them:
        // 47 instructions a step against 65
        const double h2 = dt * 0.5, h6 = dt / 6.0;
        double a, b, d, w;
        asm volatile(LZ_STEP_LOOP(60, 47,
                         LZ_QUAD_FIELD("56", "57", "%[a]")
                         "v_mul_f64 v[58:59], %[a], %[h2]\n"
                         "v_add_f64 v[58:59], v[56:57], v[58:59]\n"
                         LZ_QUAD_FIELD("58", "59", "%[b]")
                         "v_mul_f64 v[58:59], %[b], %[h2]\n"
                         "v_add_f64 v[58:59], v[56:57], v[58:59]\n"
                         LZ_QUAD_FIELD("58", "59", "%[t]")
                         "v_mul_f64 v[58:59], %[t], %[dt]\n"
                         "v_add_f64 v[58:59], v[56:57], v[58:59]\n"
                         "v_add_f64 %[b], %[b], %[t]\n"
                         LZ_QUAD_FIELD("58", "59", "%[d]")
                         "v_add_f64 %[a], %[a], %[d]\n"
                         "v_fma_f64 %[a], 2.0, %[b], %[a]\n"
                         "v_mul_f64 %[a], %[a], %[h6]\n"
                         "v_add_f64 v[56:57], v[56:57], %[a]\n")
                     : "+{v[56:57]}"(v), "=&{v[58:59]}"(w), "=&{v[60:61]}"(p1), "=&{v[62:63]}"(p2), [q0] "=&v"(q0),
                       [u] "=&v"(u), [t] "=&v"(t), [a] "=&v"(a), [b] "=&v"(b), [d] "=&v"(d), [q] "+s"(n.q)
                     : [at] "s"(n.at), [m] "v"(role.m), [c] "v"(role.c), [k] "v"(role.k), [s] "v"(role.s), [dt] "s"(dt), [h2] "v"(h2),
                       [h6] "v"(h6)
                     : LZ_STEP_CLOBBER);
    } else {
        static_assert(I == LZ_INTEGRATOR_EULER, "the quad form of this integrator is no shorter than the one-lane form");
        asm volatile(LZ_STEP_LOOP(120, 11,
                         LZ_QUAD_FIELD("56", "57", "%[t]")
                         "v_mul_f64 %[t], %[t], %[dt]\n"
                         "v_add_f64 v[56:57], v[56:57], %[t]\n")
                     : "+{v[56:57]}"(v), "=&{v[60:61]}"(p1), "=&{v[62:63]}"(p2), [q0] "=&v"(q0), [u] "=&v"(u),
                       [t] "=&v"(t), [q] "+s"(n.q)
                     : [at] "s"(n.at), [m] "v"(role.m), [c] "v"(role.c), [k] "v"(role.k), [s] "v"(role.s), [dt] "s"(dt)
                     : LZ_STEP_CLOBBER);
    }
    x = dpp_f64<0x00>(v);  // quad_perm [0,0,0,0], [1,1,1,1], [2,2,2,2]
    y = dpp_f64<0x55>(v);
    z = dpp_f64<0xAA>(v);
}

// ---- one chain over a row of 16 lanes -------------------------------------------------
//
// A row's binary64 instruction can read one lane of the row in all lanes (row_newbcast), so an
// increment travels and is added in one v_fmac_f64, where a quad needs two moves and the addition.
// Bank 0 (lanes 0-3 of the row) computes x, bank 1 y, bank 2 z; bank 3 holds zeros.  Each bank keeps
// what it needs of the coordinates, all advanced by the same increments t = dt (dx, dy, dz) and so
// equal to the last bit:
//
//     w  = (x, y, z)      s1 = (y, z, y)      c = (sigma, x, x)      s2 = (-x, rho, 0)
//     t = s s1 + s2       (y - x, rho - z, y)          w  += t
//     t = t c             (sigma (y-x), x (rho-z), xy) s2 -= t                  bank 0
//     t = t - u           (dx, dy, dz)                 s1 += t of bank 1        banks 0, 2
//     t = t dt                                         c  += t of bank 0        banks 1, 2
//                                                      u   = (0, y, beta z)
//                                                      s1 += t of bank 2        bank 1
//
// 10 instructions (8 for the fused Euler map, whose increments carry dt in the v_fmac_f64) in this order,
// which keeps two instructions between a write and a DPP instruction that reads it, s1's two
// masked additions among them.  Measured with one wave per SIMD: 40.6 clocks per step, against 44.6 in a quad.  A
// wave holds 4 chains.
//
// RK4 takes the quad's field with each bank's coordinate in v: a 64-bit move of a broadcast, masked to the banks that read
// it, takes the place of a quad's two 32-bit moves, and P1 comes in two of them (y for banks 0 and 2, z for bank 1), so
// a field is 8 instructions and a step 43, 173.5 clocks against 190.

// The vector field of the value V into OUT, banks as lanes of a quad (see LZ_QUAD_FIELD).
#define LZ_ROW_FIELD(V, OUT)                                                                   \
    "v_fma_f64 %[q0], %[m], " V ", %[c]\n"                                                     \
    "v_mul_f64 %[u], %[k], " V "\n"                                                            \
    "v_mov_b64_dpp %[p1], " V " row_newbcast:4 row_mask:0xf bank_mask:0x5\n"                   \
    "v_mov_b64_dpp %[p2], " V " row_newbcast:0 row_mask:0xf bank_mask:0x6\n"                   \
    "v_mov_b64_dpp %[p1], " V " row_newbcast:8 row_mask:0xf bank_mask:0x2\n"                   \
    "v_fma_f64 " OUT ", %[s], %[p1], %[q0]\n"                                                  \
    "v_mul_f64 " OUT ", " OUT ", %[p2]\n"                                                      \
    "v_add_f64 " OUT ", " OUT ", -%[u]\n"

template <int I>
__device__ __forceinline__ void row_steps(double &x, double &y, double &z, double dt, uint32_t n_it,
                                          const LaneRole<16> &role, int lane) {
    const int r = (lane >> 2) & 3;
    double w = r == 0 ? x : (r == 1 ? y : (r == 2 ? z : 0.0));
    if constexpr (I == LZ_INTEGRATOR_RK4) {
        const double h2 = dt * 0.5, h6 = dt / 6.0, c = r == 1 ? RHO : 0.0;
        double p1 = 0.0, p2 = r == 0 ? SIGMA : 0.0, q0, u, a, b, d, e, v;
        StepCount n(n_it, RK4_U, 43);
        asm volatile(LZ_STEP_LOOP(60, 43,
                         LZ_ROW_FIELD("%[w]", "%[a]")
                         "v_mul_f64 %[v], %[a], %[h2]\n"
                         "v_add_f64 %[v], %[w], %[v]\n"
                         LZ_ROW_FIELD("%[v]", "%[b]")
                         "v_mul_f64 %[v], %[b], %[h2]\n"
                         "v_add_f64 %[v], %[w], %[v]\n"
                         LZ_ROW_FIELD("%[v]", "%[e]")
                         "v_mul_f64 %[v], %[e], %[dt]\n"
                         "v_add_f64 %[v], %[w], %[v]\n"
                         "v_add_f64 %[b], %[b], %[e]\n"
                         LZ_ROW_FIELD("%[v]", "%[d]")
                         "v_add_f64 %[a], %[a], %[d]\n"
                         "v_fma_f64 %[a], 2.0, %[b], %[a]\n"
                         "v_mul_f64 %[a], %[a], %[h6]\n"
                         "v_add_f64 %[w], %[w], %[a]\n")
                     : [w] "+v"(w), [p1] "+v"(p1), [p2] "+v"(p2), [q0] "=&v"(q0), [u] "=&v"(u), [a] "=&v"(a), [b] "=&v"(b),
                       [d] "=&v"(d), [e] "=&v"(e), [v] "=&v"(v), [q] "+s"(n.q)
                     : [at] "s"(n.at), [m] "v"(role.m), [c] "v"(c), [k] "v"(role.k), [s] "v"(role.s), [dt] "v"(dt), [h2] "v"(h2), [h6] "v"(h6)
                     : LZ_STEP_CLOBBER);
        x = dpp_f64<0x150>(w);  // row_newbcast of lanes 0, 4, 8
        y = dpp_f64<0x154>(w);
        z = dpp_f64<0x158>(w);
        return;
    }
    double s1 = r == 1 ? z : (r == 3 ? 0.0 : y);
    double c = r == 0 ? SIGMA : (r == 3 ? 0.0 : x);
    double s2 = r == 0 ? -x : (r == 1 ? RHO : 0.0);
    double u = role.k * w, t;
    StepCount n(n_it, STEP_U, I == LZ_INTEGRATOR_EULER_FMA ? 8 : 10);
    if constexpr (I == LZ_INTEGRATOR_EULER_FMA) {
        const double dtv = dt, mdt = role.m * dt;
        asm volatile(LZ_STEP_LOOP(120, 8,
                         "v_fma_f64 %[t], %[s], %[s1], %[s2]\n"
                         "v_fma_f64 %[t], %[t], %[c], -%[u]\n"
                         "v_fma_f64 %[w], %[dt], %[t], %[w]\n"
                         "v_fma_f64 %[s2], %[mdt], %[t], %[s2]\n"
                         "v_fmac_f64_dpp %[s1], %[t], %[dt] row_newbcast:4 row_mask:0xf bank_mask:0x5\n"
                         "v_fmac_f64_dpp %[c], %[t], %[dt] row_newbcast:0 row_mask:0xf bank_mask:0x6\n"
                         "v_mul_f64 %[u], %[k], %[w]\n"
                         "v_fmac_f64_dpp %[s1], %[t], %[dt] row_newbcast:8 row_mask:0xf bank_mask:0x2\n")
                     : [w] "+v"(w), [s1] "+v"(s1), [c] "+v"(c), [s2] "+v"(s2), [u] "+v"(u), [t] "=&v"(t), [q] "+s"(n.q)
                     : [at] "s"(n.at), [k] "v"(role.k), [s] "v"(role.s), [dt] "v"(dtv), [mdt] "v"(mdt)
                     : LZ_STEP_CLOBBER);
    } else {
        asm volatile(LZ_STEP_LOOP(120, 10,
                         "v_fma_f64 %[t], %[s], %[s1], %[s2]\n"
                         "v_mul_f64 %[t], %[t], %[c]\n"
                         "v_add_f64 %[t], %[t], -%[u]\n"
                         "v_mul_f64 %[t], %[t], %[dt]\n"
                         "v_add_f64 %[w], %[w], %[t]\n"
                         "v_fma_f64 %[s2], %[m], %[t], %[s2]\n"
                         "v_fmac_f64_dpp %[s1], %[t], %[one] row_newbcast:4 row_mask:0xf bank_mask:0x5\n"
                         "v_fmac_f64_dpp %[c], %[t], %[one] row_newbcast:0 row_mask:0xf bank_mask:0x6\n"
                         "v_mul_f64 %[u], %[k], %[w]\n"
                         "v_fmac_f64_dpp %[s1], %[t], %[one] row_newbcast:8 row_mask:0xf bank_mask:0x2\n")
                     : [w] "+v"(w), [s1] "+v"(s1), [c] "+v"(c), [s2] "+v"(s2), [u] "+v"(u), [t] "=&v"(t), [q] "+s"(n.q)
                     : [at] "s"(n.at), [k] "v"(role.k), [s] "v"(role.s), [m] "v"(role.m), [one] "v"(role.one), [dt] "s"(dt)
                     : LZ_STEP_CLOBBER);
    }
    x = dpp_f64<0x150>(w);  // row_newbcast of lanes 0, 4, 8
    y = dpp_f64<0x154>(w);
    z = dpp_f64<0x158>(w);
}

// State of the M chains of one lane.
template <int M>
struct Chains {
    double x[M], y[M], z[M];     // r
    double a0[M], a1[M], a2[M];  // alpha
    uint32_t mu0[M], mu1[M], mu2[M];
    uint32_t om0[M], om1[M], om2[M];
    double ap0[M], ap1[M], ap2[M];  // a'
    uint32_t k0[M], k1[M], k2[M];
    uint32_t dec[M];                // 1 = decrypt
};

// Block b starts at r0 + b 2^-24 (every coordinate); alpha_i = r[mu_i] (Eq. alpha, n = 0).
template <int M>
__device__ __forceinline__ void init_chain(Chains<M> &c, int m, const double (&r0)[3], const double (&ap)[3],
                                           const uint8_t (&mu)[3], const uint8_t (&om)[3], const uint8_t (&k)[3],
                                           uint64_t b, uint32_t dec) {
    const double off = (double)b * 0x1p-24;
    c.x[m] = r0[0] + off;
    c.y[m] = r0[1] + off;
    c.z[m] = r0[2] + off;
    c.mu0[m] = mu[0]; c.mu1[m] = mu[1]; c.mu2[m] = mu[2];
    c.om0[m] = om[0]; c.om1[m] = om[1]; c.om2[m] = om[2];
    c.a0[m] = sel3(c.mu0[m], c.x[m], c.y[m], c.z[m]);
    c.a1[m] = sel3(c.mu1[m], c.x[m], c.y[m], c.z[m]);
    c.a2[m] = sel3(c.mu2[m], c.x[m], c.y[m], c.z[m]);
    c.ap0[m] = ap[0]; c.ap1[m] = ap[1]; c.ap2[m] = ap[2];
    c.k0[m] = k[0]; c.k1[m] = k[1]; c.k2[m] = k[2];
    c.dec[m] = dec;
}

__device__ __forceinline__ uint32_t mod_k(uint32_t v, uint32_t k) { return k == 4 ? (v & 3u) : v % 3u; }

// Steps 1-3 of Section 3.2 for one byte of each of the M chains.
template <int M, int I, int G>
__device__ __forceinline__ void crypt_byte(Chains<M> &c, const uint32_t (&bin)[M], uint32_t (&bout)[M], double dt,
                                           uint32_t n_it, const LaneRole<G> &role, int lane) {
    uint32_t R1[M], R2[M], p[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        // Step 1: y = (x + R1 + R2) mod 2^8 (encode) or x = (y - R1 - R2) mod 2^8 (decode)
        R1[m] = r_nu(c.a0[m], c.om0[m]);
        R2[m] = r_nu(c.a1[m], c.om1[m]);
        const uint32_t ks = R1[m] + R2[m];
        if (c.dec[m]) {
            p[m] = (bin[m] - ks) & 0xFFu;
            bout[m] = p[m];
        } else {
            p[m] = bin[m];
            bout[m] = (bin[m] + ks) & 0xFFu;
        }
        // Step 2: Theta = P_i / 10^(3 + Omega_3) added to the coordinate mu_3
        const double th = theta_of(p[m], c.om2[m]);
        // r[mu_3] += Theta, written as value selects: a select of the coordinate's address
        // would force the chain state out of registers
        const uint32_t s = c.mu2[m];
        const double moved = sel3(s, c.x[m], c.y[m], c.z[m]) + th;
        c.x[m] = s == 0 ? moved : c.x[m];
        c.y[m] = s == 1 ? moved : c.y[m];
        c.z[m] = s == 2 ? moved : c.z[m];
    }
    // Step 2 (cont.): r <- F^(n_it)(r)
    if constexpr (G == 16) row_steps<I>(c.x[0], c.y[0], c.z[0], dt, n_it, role, lane);
    else if constexpr (G == 4) quad_steps<I>(c.x[0], c.y[0], c.z[0], dt, n_it, role, lane);
    else lorenz_steps<M, I>(c.x, c.y, c.z, dt, n_it);
#pragma unroll
    for (int m = 0; m < M; ++m) {
        // Step 3: mu_i <- (mu_i + R_i) mod 3 with R_i from the old alpha_i, Omega_i
        const uint32_t R3 = r_nu(c.a2[m], c.om2[m]);
        c.mu0[m] = (c.mu0[m] + R1[m]) % 3u;
        c.mu1[m] = (c.mu1[m] + R2[m]) % 3u;
        c.mu2[m] = (c.mu2[m] + R3) % 3u;
        // alpha_i = r[mu_i] (Eq. alpha), then Omega_i <- (Omega_i + R(alpha_i, Omega_i)) mod k_i
        // (the index [(i+2) mod 3]+1 evaluated 1-based is i itself)
        c.a0[m] = sel3(c.mu0[m], c.x[m], c.y[m], c.z[m]);
        c.a1[m] = sel3(c.mu1[m], c.x[m], c.y[m], c.z[m]);
        c.a2[m] = sel3(c.mu2[m], c.x[m], c.y[m], c.z[m]);
        c.om0[m] = mod_k(c.om0[m] + r_nu(c.a0[m], c.om0[m]), c.k0[m]);
        c.om1[m] = mod_k(c.om1[m] + r_nu(c.a1[m], c.om1[m]), c.k1[m]);
        c.om2[m] = mod_k(c.om2[m] + r_nu(c.a2[m], c.om2[m]), c.k2[m]);
        // r <- r + a'
        c.x[m] = c.x[m] + c.ap0[m];
        c.y[m] = c.y[m] + c.ap1[m];
        c.z[m] = c.z[m] + c.ap2[m];
    }
}

// ---- wave-level helpers -------------------------------------------------------------

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)v, off, WAVE);
        v = o > v ? o : v;
    }
    return v;
}

__device__ __forceinline__ unsigned long long wave_xor_u64(unsigned long long v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, off, WAVE);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), off, WAVE);
        v ^= ((unsigned long long)hi << 32) | lo;
    }
    return v;
}

// Per-wave LDS layout: tile rows (one per chain of the wave x stride), then the chain table.
struct WaveLds {
    uint8_t *tile;
    const uint8_t **in;
    uint8_t **out;
    uint32_t *cnt;
};

// Row stride of the LDS tile: an odd number of 4-byte words past a multiple of 64 banks
// (tile is a multiple of 16), so the 64 lanes reading their own rows hit distinct banks.
__host__ __device__ constexpr size_t tile_stride(int tile) { return (size_t)tile + 4; }
__host__ __device__ constexpr size_t wave_lds_bytes(int rows, int tile) {
    return (size_t)rows * (tile_stride(tile) + 2 * sizeof(void *) + sizeof(uint32_t));
}

template <int ROWS>
__device__ __forceinline__ WaveLds wave_lds(char *base, int tile) {
    WaveLds w;
    w.tile = reinterpret_cast<uint8_t *>(base);
    char *p = base + (size_t)ROWS * tile_stride(tile);
    w.in = reinterpret_cast<const uint8_t **>(p);
    p += (size_t)ROWS * sizeof(void *);
    w.out = reinterpret_cast<uint8_t **>(p);
    p += (size_t)ROWS * sizeof(void *);
    w.cnt = reinterpret_cast<uint32_t *>(p);
    return w;
}

// Runs cnt[m] bytes of every chain of the wave through crypt_byte, staging
// input and output through LDS.  on_stop(m) is called right after chain m's
// last byte (or before the loop when cnt[m] == 0), with c holding that chain's
// state; chains past their end keep running on zero bytes but their results
// are neither stored nor used.  G lanes hold the same chain and the same arguments; they write the
// same bytes to its row, and on_stop runs in each of them.
template <int M, int I, int G, typename OnStop>
__device__ __forceinline__ void wave_run(Chains<M> &c, const WaveLds &w, int tile, const uint8_t *const (&in)[M],
                                         uint8_t *const (&out)[M], const uint32_t (&cnt)[M], double dt,
                                         uint32_t n_it, int lane, OnStop on_stop) {
    static_assert(G == 1 || M == 1, "a chain over several lanes is one chain per lane group");
    const LaneRole<G> role(lane);
    const int ch = lane / G;  // the lane's chain among the wave's (row m * WAVE + ch)
    uint32_t mx = 0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        w.in[m * WAVE + ch] = in[m];
        w.out[m * WAVE + ch] = out[m];
        w.cnt[m * WAVE + ch] = cnt[m];
        mx = cnt[m] > mx ? cnt[m] : mx;
        if (cnt[m] == 0) on_stop(m);
    }
    mx = wave_max_u32(mx);
    wave_sync();
    const size_t stride = tile_stride(tile);
    constexpr int rows = WAVE * M / G;
    for (uint32_t t0 = 0; t0 < mx; t0 += (uint32_t)tile) {
        // stage in: byte u of the wave tile -> row u / tile, column u % tile
        for (int u = lane; u < rows * tile; u += WAVE) {
            const int row = u / tile, col = u % tile;
            const uint32_t j = t0 + (uint32_t)col;
            if (j < w.cnt[row]) w.tile[row * stride + col] = w.in[row][j];
        }
        wave_sync();
        const uint32_t nk = mx - t0 < (uint32_t)tile ? mx - t0 : (uint32_t)tile;
        for (uint32_t kk = 0; kk < nk; ++kk) {
            const uint32_t j = t0 + kk;
            uint32_t bin[M], bout[M];
#pragma unroll
            for (int m = 0; m < M; ++m) bin[m] = j < cnt[m] ? w.tile[(m * WAVE + ch) * stride + kk] : 0u;
            crypt_byte<M, I, G>(c, bin, bout, dt, n_it, role, lane);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                if (j < cnt[m]) w.tile[(m * WAVE + ch) * stride + kk] = (uint8_t)bout[m];
                if (j + 1 == cnt[m]) on_stop(m);
            }
        }
        wave_sync();
        // stage out
        for (int u = lane; u < rows * tile; u += WAVE) {
            const int row = u / tile, col = u % tile;
            const uint32_t j = t0 + (uint32_t)col;
            if (j < w.cnt[row]) w.out[row][j] = w.tile[row * stride + col];
        }
        wave_sync();
    }
}

// ---- room for wide launches ------------------------------------------------------------
//
// Spreading chains over lanes costs more instructions per chain in all (3.2 times as many at G = 4, 11.5
// times at G = 16), which is free only on SIMDs that would idle.  A launch that may run wide is preceded by claim_kernel, which adds
// its waves to the device's count of waves in flight and lets it run wide if all of them together are
// at most one per SIMD; otherwise the launch runs one chain per lane (the waves it then does not need
// end at once).  Calls that overlap on several streams so take the idle SIMDs first and then run as
// densely as before, whatever runs beside them: every kernel of the cipher counts its waves, and a call of several
// rounds holds its claim from before the first to the end of the last.
__device__ uint32_t g_waves;

// Adds the waves of a workgroup that no claim counted (n > 0) or takes them off at its end (n < 0).
__device__ __forceinline__ void count_waves(int n) {
    if (threadIdx.x == 0) atomicAdd(&g_waves, (uint32_t)n);
}

// Clears n words (the tag accumulators), and decides whether the launch of `waves` waves that
// follows on the stream runs wide: *wide = 1 or 0.
__global__ void claim_kernel(unsigned long long *p, size_t n, unsigned long long *wide, uint32_t waves, uint32_t simds) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = t; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
    if (t == 0) *wide = atomicAdd(&g_waves, waves) + waves <= simds ? 1 : 0;
}

// Takes off the waves of a launch that was claimed for and then refused.
__global__ void give_back_kernel(uint32_t waves, const unsigned long long *wide) {
    if (!wide || *wide) atomicSub(&g_waves, waves);
}

// ---- plain path: one message ---------------------------------------------------------

struct PlainArgs {
    double ap[3], r0[3];
    uint8_t mu[3], om[3], k[3];
    uint32_t decrypt;
    double dt;
    uint32_t n_it, block_len, tile;
    const uint8_t *in;
    uint8_t *out;
    uint64_t n, nb;
    uint64_t block_base;  // index of the first block (0 for a whole message)
    unsigned long long *tag_acc;
    const unsigned long long *wide;  // G > 1: claim_kernel's answer
    StreamExtra x;        // read only by the stream instance (X = true)
};

__device__ __forceinline__ void load_slot(Chains<1> &c, const ChainSlot &s, const double (&ap)[3],
                                          const uint8_t (&k)[3], uint32_t dec) {
    c.x[0] = s.r[0]; c.y[0] = s.r[1]; c.z[0] = s.r[2];
    c.a0[0] = s.al[0]; c.a1[0] = s.al[1]; c.a2[0] = s.al[2];
    c.mu0[0] = s.mu[0]; c.mu1[0] = s.mu[1]; c.mu2[0] = s.mu[2];
    c.om0[0] = s.om[0]; c.om1[0] = s.om[1]; c.om2[0] = s.om[2];
    c.ap0[0] = ap[0]; c.ap1[0] = ap[1]; c.ap2[0] = ap[2];
    c.k0[0] = k[0]; c.k1[0] = k[1]; c.k2[0] = k[2];
    c.dec[0] = dec;
}

__device__ __forceinline__ void save_slot(ChainSlot &s, const Chains<1> &c) {
    s.r[0] = c.x[0]; s.r[1] = c.y[0]; s.r[2] = c.z[0];
    s.al[0] = c.a0[0]; s.al[1] = c.a1[0]; s.al[2] = c.a2[0];
    s.mu[0] = (uint8_t)c.mu0[0]; s.mu[1] = (uint8_t)c.mu1[0]; s.mu[2] = (uint8_t)c.mu2[0];
    s.om[0] = (uint8_t)c.om0[0]; s.om[1] = (uint8_t)c.om1[0]; s.om[2] = (uint8_t)c.om2[0];
}

// X: the stream instance (M = 1), whose chains nb and nb + 1 may be a.x's head and tail.  G lanes
// carry each chain.
template <int M, int I, bool X, int G>
__device__ __forceinline__ void plain_body(const PlainArgs &a, char *lds) {
    static_assert(!X || M == 1, "the stream instance runs one chain per lane group");
    constexpr int ROWS = WAVE * M / G;
    const int lane = threadIdx.x % WAVE;
    const int wid = threadIdx.x / WAVE;
    const int wpw = blockDim.x / WAVE;
    const WaveLds w = wave_lds<ROWS>(lds + (size_t)wid * wave_lds_bytes(ROWS, a.tile), a.tile);
    const uint64_t base = ((uint64_t)blockIdx.x * wpw + wid) * ROWS;
    if (base >= a.nb + (X ? 2 : 0)) return;  // no chain

    Chains<M> c;
    const uint8_t *in[M];
    uint8_t *out[M];
    uint32_t cnt[M];
    bool valid[M];
    unsigned long long d0[M], d1[M], d2[M];
    double r0[3] = {a.r0[0], a.r0[1], a.r0[2]}, ap[3] = {a.ap[0], a.ap[1], a.ap[2]};
    uint8_t mu[3] = {a.mu[0], a.mu[1], a.mu[2]}, om[3] = {a.om[0], a.om[1], a.om[2]},
            k[3] = {a.k[0], a.k[1], a.k[2]};
    // stream instance: 1 = this lane's chain is the head, 2 = the tail
    const uint32_t n_head = X && a.x.head_slot ? 1u : 0u;
    const uint64_t g0 = base + lane / G;
    const uint32_t role = !X || g0 < a.nb ? 0u : (g0 == a.nb && n_head ? 1u : (g0 == a.nb + n_head && a.x.tail_slot ? 2u : 0u));
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const uint64_t g = base + (uint64_t)m * WAVE + lane / G;
        valid[m] = g < a.nb;
        const uint64_t off = g * a.block_len;
        cnt[m] = (valid[m] && off < a.n) ? (uint32_t)(a.n - off < a.block_len ? a.n - off : a.block_len) : 0u;
        in[m] = a.in + (valid[m] && off < a.n ? off : 0);
        out[m] = a.out + (valid[m] && off < a.n ? off : 0);
        init_chain<M>(c, m, r0, ap, mu, om, k, a.block_base + (valid[m] ? g : 0), a.decrypt);
        d0[m] = d1[m] = d2[m] = 0;
    }
    if constexpr (X) {
        if (role == 1) {
            load_slot(c, *a.x.head_slot, ap, k, a.decrypt);
            valid[0] = a.x.head_complete != 0;
            cnt[0] = a.x.head_cnt;
            in[0] = a.x.head_in;
            out[0] = a.x.head_out;
        } else if (role == 2) {
            init_chain<1>(c, 0, r0, ap, mu, om, k, a.x.tail_block, a.decrypt);
            cnt[0] = a.x.tail_cnt;
            in[0] = a.x.tail_in;
            out[0] = a.x.tail_out;
        }
    }
    wave_run<M, I, G>(c, w, (int)a.tile, in, out, cnt, a.dt, a.n_it, lane, [&](int m) __attribute__((always_inline)) {
        if constexpr (X) {
            if (role == 2 || (role == 1 && !a.x.head_complete)) {
                save_slot(role == 2 ? *a.x.tail_slot : *a.x.head_slot, c);
                return;
            }
        }
        d0[m] = digest_word(c.x[m]);
        d1[m] = digest_word(c.y[m]);
        d2[m] = digest_word(c.z[m]);
    });
    unsigned long long t0 = 0, t1 = 0, t2 = 0;
#pragma unroll
    for (int m = 0; m < M; ++m)
        if (valid[m] && lane % G == 0) { t0 ^= d0[m]; t1 ^= d1[m]; t2 ^= d2[m]; }
    t0 = wave_xor_u64(t0);
    t1 = wave_xor_u64(t1);
    t2 = wave_xor_u64(t2);
    if (lane == 0) {
        atomicXor(&a.tag_acc[0], t0);
        atomicXor(&a.tag_acc[1], t1);
        atomicXor(&a.tag_acc[2], t2);
    }
}

template <int M, int I, bool X, int G>
__global__ __launch_bounds__(256) void plain_kernel(PlainArgs a) {
    extern __shared__ char lds[];
    const int waves = blockDim.x / WAVE;
    if constexpr (G == 1) {
        count_waves(waves);
        plain_body<M, I, X, 1>(a, lds);
    } else {
        if (*a.wide) plain_body<M, I, X, G>(a, lds);
        else plain_body<M, I, X, 1>(a, lds);
    }
    count_waves(-waves);
}

// The rounds' waves are counted by a claim before the launch that comes first, to the end of the last round.
__device__ __forceinline__ void seg_done(const SegPlan &p, uint64_t first) {
    const int waves = blockDim.x / WAVE;
    if (first + (uint64_t)gridDim.x * waves >= p.off[p.segs]) count_waves(-waves);
}

// One round of a segment plan (see plan_segments): each wave advances 64 chains by one segment of
// seg_len bytes from the checkpoint that an earlier round left.  The round's waves are tasks
// first, first + 1, ... of the plan; task off[s] + w is segment s of wave w.
__device__ __forceinline__ bool seg_task(const SegPlan &p, uint64_t first, uint32_t &seg, uint32_t &wave) {
    const uint64_t t = first + (uint64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
    if (t >= p.off[p.segs]) return false;
    seg = 0;
    while (t >= p.off[seg + 1]) ++seg;
    wave = (uint32_t)(t - p.off[seg]);
    return true;
}

// Runs cnt bytes of the lanes' chain from byte pos of its block of len bytes: from its start (pos = 0, c
// initialised by the caller) or from `st`, to its end (then d holds the digest and the result is true in
// the chain's first lane) or back to `st`.  A lane with cnt = 0 has nothing left to do.
__device__ __forceinline__ void load_state(Chains<1> &c, const ChainState &s) {
    c.x[0] = s.r[0]; c.y[0] = s.r[1]; c.z[0] = s.r[2];
    c.a0[0] = s.al[0]; c.a1[0] = s.al[1]; c.a2[0] = s.al[2];
    c.mu0[0] = s.mu[0]; c.mu1[0] = s.mu[1]; c.mu2[0] = s.mu[2];
    c.om0[0] = s.om[0]; c.om1[0] = s.om[1]; c.om2[0] = s.om[2];
}

__device__ __forceinline__ void save_state(ChainState &s, const Chains<1> &c) {
    s.r[0] = c.x[0]; s.r[1] = c.y[0]; s.r[2] = c.z[0];
    s.al[0] = c.a0[0]; s.al[1] = c.a1[0]; s.al[2] = c.a2[0];
    s.mu[0] = (uint8_t)c.mu0[0]; s.mu[1] = (uint8_t)c.mu1[0]; s.mu[2] = (uint8_t)c.mu2[0];
    s.om[0] = (uint8_t)c.om0[0]; s.om[1] = (uint8_t)c.om1[0]; s.om[2] = (uint8_t)c.om2[0];
}

template <int I, int G = 1>
__device__ __forceinline__ bool seg_run(Chains<1> &c, const WaveLds &w, uint32_t tile, const uint8_t *in, uint8_t *out,
                                        uint32_t pos, uint32_t cnt, uint32_t len, ChainState &st, double dt,
                                        uint32_t n_it, int lane, unsigned long long (&d)[3]) {
    if (pos > 0 && cnt > 0) load_state(c, st);
    const uint8_t *ins[1] = {in};
    uint8_t *outs[1] = {out};
    const uint32_t cnts[1] = {cnt};
    wave_run<1, I, G>(c, w, (int)tile, ins, outs, cnts, dt, n_it, lane, [&](int) __attribute__((always_inline)) {
        if (cnt == 0) return;
        if (pos + cnt == len) {
            d[0] = digest_word(c.x[0]);
            d[1] = digest_word(c.y[0]);
            d[2] = digest_word(c.z[0]);
        } else {
            save_state(st, c);
        }
    });
    return cnt > 0 && pos + cnt == len && lane % G == 0;
}

template <int I>
__global__ __launch_bounds__(256) void plain_seg_kernel(PlainArgs a, SegPlan p, uint64_t first) {
    extern __shared__ char lds[];
    const int lane = threadIdx.x % WAVE;
    uint32_t seg, wave;
    if (seg_task(p, first, seg, wave)) {
        const WaveLds w = wave_lds<WAVE>(lds + (size_t)(threadIdx.x / WAVE) * wave_lds_bytes(WAVE, a.tile), a.tile);
        const uint64_t i = (uint64_t)wave * WAVE + lane, g = p.chain0 + i, off = g * a.block_len;
        const uint32_t len = g < a.nb ? (uint32_t)(a.n - off < a.block_len ? a.n - off : a.block_len) : 0u;
        const uint32_t pos = seg * p.seg_len;
        const uint32_t cnt = pos < len ? (len - pos < p.seg_len ? len - pos : p.seg_len) : 0u;
        const uint64_t at = cnt ? off + pos : 0;
        Chains<1> c;
        const double r0[3] = {a.r0[0], a.r0[1], a.r0[2]}, ap[3] = {a.ap[0], a.ap[1], a.ap[2]};
        const uint8_t mu[3] = {a.mu[0], a.mu[1], a.mu[2]}, om[3] = {a.om[0], a.om[1], a.om[2]},
                      k[3] = {a.k[0], a.k[1], a.k[2]};
        init_chain<1>(c, 0, r0, ap, mu, om, k, a.block_base + (g < a.nb ? g : 0), a.decrypt);
        unsigned long long d[3] = {0, 0, 0};
        const bool done = seg_run<I>(c, w, a.tile, a.in + at, a.out + at, pos, cnt, len, p.state[i], a.dt, a.n_it, lane, d);
        if (__any(done)) {
            const unsigned long long t0 = wave_xor_u64(done ? d[0] : 0ull), t1 = wave_xor_u64(done ? d[1] : 0ull),
                                     t2 = wave_xor_u64(done ? d[2] : 0ull);
            if (lane == 0) {
                atomicXor(&a.tag_acc[0], t0);
                atomicXor(&a.tag_acc[1], t1);
                atomicXor(&a.tag_acc[2], t2);
            }
        }
    }
    seg_done(p, first);
}

// The byte that a unit of a mix plan starts a round at: it has run n times in GA lanes before round r, n the
// multiples u, u + U, ... below r A, so its position follows from r alone.
__device__ __forceinline__ uint32_t mix_pos(const MixPlan &p, uint32_t round, uint32_t unit) {
    const uint32_t ra = round * p.a, n = ra > unit ? (ra - 1 - unit) / p.units + 1 : 0;
    return n * p.la + (round - n) * p.lb;
}

// One round of a mix plan (see plan_mix): the chains of one unit, in GA lanes each (`first` = 0) or a quarter or
// sixteenth of them in GB, advance by la or lb bytes.
template <int I, bool X, int G>
__device__ __forceinline__ void mix_body(const PlainArgs &a, const MixPlan &p, uint32_t round, uint32_t unit,
                                         uint32_t first, uint32_t step, char *lds) {
    constexpr int ROWS = WAVE / G;
    const int lane = threadIdx.x % WAVE;
    const WaveLds w = wave_lds<ROWS>(lds + (size_t)(threadIdx.x / WAVE) * wave_lds_bytes(WAVE, a.tile), a.tile);
    const uint32_t pos = mix_pos(p, round, unit);
    const uint64_t g = (uint64_t)unit * p.unit + first + lane / G, off = g * a.block_len;
    const uint32_t n_head = X && a.x.head_slot ? 1u : 0u;
    const uint32_t role = !X || g < a.nb ? 0u : (g == a.nb && n_head ? 1u : (g == a.nb + n_head && a.x.tail_slot ? 2u : 0u));
    uint32_t len = g < a.nb ? (uint32_t)(a.n - off < a.block_len ? a.n - off : a.block_len) : 0u;
    const uint8_t *in = a.in + (g < a.nb ? off : 0);
    uint8_t *out = a.out + (g < a.nb ? off : 0);
    const double r0[3] = {a.r0[0], a.r0[1], a.r0[2]}, ap[3] = {a.ap[0], a.ap[1], a.ap[2]};
    const uint8_t mu[3] = {a.mu[0], a.mu[1], a.mu[2]}, om[3] = {a.om[0], a.om[1], a.om[2]},
                  k[3] = {a.k[0], a.k[1], a.k[2]};
    uint64_t block = a.block_base + (g < a.nb ? g : 0);
    if constexpr (X) {
        if (role == 1) {
            len = a.x.head_cnt;
            in = a.x.head_in;
            out = a.x.head_out;
        } else if (role == 2) {
            len = a.x.tail_cnt;
            in = a.x.tail_in;
            out = a.x.tail_out;
            block = a.x.tail_block;
        }
    }
    const uint32_t cnt = pos < len ? (len - pos < step ? len - pos : step) : 0u;
    Chains<1> c;
    init_chain<1>(c, 0, r0, ap, mu, om, k, block, a.decrypt);
    if (cnt) {
        in += pos;
        out += pos;
        if (pos > 0) load_state(c, p.state[g]);
        else if (X && role == 1) load_slot(c, *a.x.head_slot, ap, k, a.decrypt);
    }
    bool done = false;
    unsigned long long d0 = 0, d1 = 0, d2 = 0;
    const uint8_t *ins[1] = {in};
    uint8_t *outs[1] = {out};
    const uint32_t cnts[1] = {cnt};
    wave_run<1, I, G>(c, w, (int)a.tile, ins, outs, cnts, a.dt, a.n_it, lane, [&](int) __attribute__((always_inline)) {
        if (cnt == 0) return;
        if (pos + cnt != len) {
            save_state(p.state[g], c);
            return;
        }
        if constexpr (X) {
            if (role == 2 || (role == 1 && !a.x.head_complete)) {
                save_slot(role == 2 ? *a.x.tail_slot : *a.x.head_slot, c);
                return;
            }
        }
        done = lane % G == 0;
        d0 = digest_word(c.x[0]);
        d1 = digest_word(c.y[0]);
        d2 = digest_word(c.z[0]);
    });
    if (__any(done)) {
        const unsigned long long t0 = wave_xor_u64(done ? d0 : 0ull), t1 = wave_xor_u64(done ? d1 : 0ull),
                                 t2 = wave_xor_u64(done ? d2 : 0ull);
        if (lane == 0) {
            atomicXor(&a.tag_acc[0], t0);
            atomicXor(&a.tag_acc[1], t1);
            atomicXor(&a.tag_acc[2], t2);
        }
    }
}

// Waves 0 .. p.a - 1 take the round's units in GA lanes, the others the rest of the units in GB, GB / GA waves a
// unit: body(lanes, unit, first chain of the unit, bytes).  The claim is held to the end of the last round, or a
// claim that comes between two rounds would be granted the SIMDs that the next one takes.  Without room on the device (claim_kernel) the
// first round runs everything, one chain per lane: all().
template <int GA, int GB, class Body, class All>
__device__ __forceinline__ void mix_round(const MixPlan &p, uint32_t round, uint32_t wide, Body &&body, All &&all) {
    const int waves = blockDim.x / WAVE;
    if (wide) {
        constexpr uint32_t K = GB / GA;
        const uint32_t v = __builtin_amdgcn_readfirstlane(blockIdx.x * waves + threadIdx.x / WAVE);
        const uint32_t start = (round * p.a) % p.units;
        if (v < p.a) {
            body(std::integral_constant<int, GA>{}, (start + v) % p.units, 0u, p.la);
        } else if ((v - p.a) / K < p.units - p.a) {
            body(std::integral_constant<int, GB>{}, (start + p.a + (v - p.a) / K) % p.units, (v - p.a) % K * (WAVE / GB), p.lb);
        }
        if (round + 1 == p.rounds) count_waves(-waves);  // claimed for all rounds, which have the same workgroups
    } else if (round == 0) {
        all();
        count_waves(-waves);
    }
}

template <int I, bool X, int GA, int GB>
__global__ __launch_bounds__(256) void mix_kernel(PlainArgs a, MixPlan p, uint32_t round) {
    extern __shared__ char lds[];
    mix_round<GA, GB>(
        p, round, *a.wide,
        [&](auto g, uint32_t unit, uint32_t first, uint32_t step) __attribute__((always_inline)) {
            mix_body<I, X, decltype(g)::value>(a, p, round, unit, first, step, lds);
        },
        [&]() __attribute__((always_inline)) { plain_body<1, I, X, 1>(a, lds); });
}

// Encrypt: tag bytes to out_tag.  Decrypt: compare with stored tag, status,
// and zero the body on failure (grid-stride over the body).
__global__ void plain_finalize_kernel(int decrypt, const unsigned long long *tag_acc, const uint8_t *stored,
                                      uint8_t *tag_out, int32_t *status, uint8_t *body, uint64_t n) {
    const unsigned long long t[3] = {tag_acc[0], tag_acc[1], tag_acc[2]};
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (!decrypt) {
        if (tid < LZ_TAG_BYTES) tag_out[tid] = (uint8_t)(t[tid / 8] >> (8 * (tid % 8)));
        return;
    }
    bool ok = true;
    for (int q = 0; q < LZ_TAG_BYTES; ++q) ok = ok && stored[q] == (uint8_t)(t[q / 8] >> (8 * (q % 8)));
    if (tid == 0 && status) *status = ok ? LZ_OK : LZ_E_INTEGRITY;
    if (!ok)
        for (uint64_t i = tid; i < n; i += (uint64_t)gridDim.x * blockDim.x) body[i] = 0;
}

// Stores the address of a batch's status array in its slot (read by batch_finalize_kernel).
__global__ void set_status_ref_kernel(int32_t **slot, int32_t *status) { *slot = status; }

__global__ void fill_u64_kernel(unsigned long long *p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// ---- batched path: persistent kernel over a work queue --------------------------------

struct BatchArgs {
    BatchDev b;
    double dt;
    uint32_t n_it, block_len, tile;
    uint64_t n_chains;  // of the persistent launch (the rest belong to a segment plan)
};

__device__ __forceinline__ uint32_t find_msg(const uint64_t *prefix, uint32_t n_msg, uint64_t g) {
    // largest i with prefix[i] <= g (prefix is non-decreasing, prefix[0] = 0)
    uint32_t lo = 0, hi = n_msg;  // invariant: prefix[lo] <= g < prefix[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Chain g of the batch: message i, block b of len bytes.
__device__ __forceinline__ void batch_chain(const BatchArgs &a, uint64_t g, uint32_t &i, uint64_t &b, uint32_t &len) {
    if (g < a.b.n_full) {
        i = find_msg(a.b.full_prefix, a.b.n_msg, g);
        b = g - a.b.full_prefix[i];
        len = a.block_len;
    } else {
        i = a.b.tail_msg[g - a.b.n_full];
        b = a.b.msgs[i].nb - 1;
        len = (uint32_t)(a.b.msgs[i].n - b * a.block_len);
    }
}

template <int M, int I, int G>
__device__ __forceinline__ void batch_body(const BatchArgs &a, char *lds) {
    constexpr int ROWS = WAVE * M / G;
    const int lane = threadIdx.x % WAVE;
    const int wid = threadIdx.x / WAVE;
    const WaveLds w = wave_lds<ROWS>(lds + (size_t)wid * wave_lds_bytes(ROWS, a.tile), a.tile);
    const uint64_t per_task = ROWS;
    const uint64_t n_chains = a.n_chains;
    const uint64_t n_tasks = (n_chains + per_task - 1) / per_task;

    // No lane-conditional region may sit inside this loop: the compiler is free to merge such
    // regions across the back edge, which leaves lanes re-entering the loop without the others.
    // Every lane therefore takes part in the task grab (lane 0 adds 1, the others 0) and in the
    // tag update (a lane past the end, or not the first of its chain's lanes, XORs 0).
    for (;;) {
        const unsigned long long grab = atomicAdd(a.b.counter, lane == 0 ? 1ull : 0ull);
        const unsigned long long task =
            ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(grab >> 32)) << 32) |
            __builtin_amdgcn_readfirstlane((uint32_t)grab);
        if (task >= n_tasks) break;

        Chains<M> c;
        const uint8_t *in[M];
        uint8_t *out[M];
        uint32_t cnt[M], msg[M];
        bool valid[M];
        unsigned long long d0[M], d1[M], d2[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const uint64_t g = task * per_task + (uint64_t)m * WAVE + lane / G;
            valid[m] = g < n_chains;
            uint32_t i = 0;
            uint64_t b = 0;
            uint32_t len = 0;
            if (valid[m]) batch_chain(a, g, i, b, len);
            const MsgDesc &md = a.b.msgs[i];
            msg[m] = i;
            cnt[m] = valid[m] ? len : 0u;
            in[m] = md.in + b * a.block_len;
            out[m] = md.out + b * a.block_len;
            const double r0[3] = {md.r0[0], md.r0[1], md.r0[2]}, ap[3] = {md.ap[0], md.ap[1], md.ap[2]};
            const uint8_t mu[3] = {md.mu[0], md.mu[1], md.mu[2]}, om[3] = {md.om[0], md.om[1], md.om[2]},
                          k[3] = {md.k[0], md.k[1], md.k[2]};
            init_chain<M>(c, m, r0, ap, mu, om, k, b, md.decrypt);
            d0[m] = d1[m] = d2[m] = 0;
        }
        wave_run<M, I, G>(c, w, (int)a.tile, in, out, cnt, a.dt, a.n_it, lane, [&](int m) __attribute__((always_inline)) {
            d0[m] = digest_word(c.x[m]);
            d1[m] = digest_word(c.y[m]);
            d2[m] = digest_word(c.z[m]);
        });
        // tag: XOR of block digests per message, one atomic per lane and word
#pragma unroll
        for (int m = 0; m < M; ++m) {
            unsigned long long *t = &a.b.tag_acc[3 * (size_t)msg[m]];
            const bool own = valid[m] && lane % G == 0;
            atomicXor(t + 0, own ? d0[m] : 0ull);
            atomicXor(t + 1, own ? d1[m] : 0ull);
            atomicXor(t + 2, own ? d2[m] : 0ull);
        }
    }
}

template <int M, int I, int G>
__global__ __launch_bounds__(256) void batch_kernel(BatchArgs a) {
    extern __shared__ char lds[];
    const int waves = blockDim.x / WAVE;
    if constexpr (G == 1) {
        count_waves(waves);
        batch_body<M, I, 1>(a, lds);
    } else {
        if (*a.b.wide) batch_body<M, I, G>(a, lds);
        else batch_body<M, I, 1>(a, lds);
    }
    count_waves(-waves);
}

// One round of the batch's segment plan.
template <int I>
__global__ __launch_bounds__(256) void batch_seg_kernel(BatchArgs a, SegPlan p, uint64_t first) {
    extern __shared__ char lds[];
    const int lane = threadIdx.x % WAVE;
    uint32_t seg, wave;
    if (seg_task(p, first, seg, wave)) {
        const WaveLds w = wave_lds<WAVE>(lds + (size_t)(threadIdx.x / WAVE) * wave_lds_bytes(WAVE, a.tile), a.tile);
        const uint64_t j = (uint64_t)wave * WAVE + lane, g = p.chain0 + j;
        uint32_t i = 0, len = 0;
        uint64_t b = 0;
        const bool valid = g < a.b.n_full + a.b.n_tail;
        if (valid) batch_chain(a, g, i, b, len);
        const MsgDesc &md = a.b.msgs[i];
        const uint32_t pos = seg * p.seg_len;
        const uint32_t cnt = pos < len ? (len - pos < p.seg_len ? len - pos : p.seg_len) : 0u;
        const uint64_t at = cnt ? b * a.block_len + pos : 0;
        Chains<1> c;
        const double r0[3] = {md.r0[0], md.r0[1], md.r0[2]}, ap[3] = {md.ap[0], md.ap[1], md.ap[2]};
        const uint8_t mu[3] = {md.mu[0], md.mu[1], md.mu[2]}, om[3] = {md.om[0], md.om[1], md.om[2]},
                      k[3] = {md.k[0], md.k[1], md.k[2]};
        init_chain<1>(c, 0, r0, ap, mu, om, k, b, md.decrypt);
        unsigned long long d[3] = {digest_word(c.x[0]), digest_word(c.y[0]), digest_word(c.z[0])};  // an empty message's
        bool done = seg_run<I>(c, w, a.tile, md.in + at, md.out + at, pos, cnt, len, p.state[j], a.dt, a.n_it, lane, d);
        done = done || (valid && len == 0 && seg == 0);
        if (done) {
            unsigned long long *t = &a.b.tag_acc[3 * (size_t)i];
            atomicXor(t + 0, d[0]);
            atomicXor(t + 1, d[1]);
            atomicXor(t + 2, d[2]);
        }
    }
    seg_done(p, first);
}

// One round of the batch's mix plan: mix_body over its chains.
template <int I, int G>
__device__ __forceinline__ void batch_mix_body(const BatchArgs &a, const MixPlan &p, uint32_t round, uint32_t unit,
                                               uint32_t first, uint32_t step, char *lds) {
    constexpr int ROWS = WAVE / G;
    const int lane = threadIdx.x % WAVE;
    const WaveLds w = wave_lds<ROWS>(lds + (size_t)(threadIdx.x / WAVE) * wave_lds_bytes(WAVE, a.tile), a.tile);
    const uint32_t pos = mix_pos(p, round, unit);
    const uint64_t g = (uint64_t)unit * p.unit + first + lane / G;
    uint32_t i = 0, len = 0;
    uint64_t b = 0;
    const bool valid = g < a.n_chains;
    if (valid) batch_chain(a, g, i, b, len);
    const MsgDesc &md = a.b.msgs[i];
    const uint32_t cnt = pos < len ? (len - pos < step ? len - pos : step) : 0u;
    const uint64_t at = cnt ? b * a.block_len + pos : 0;
    Chains<1> c;
    const double r0[3] = {md.r0[0], md.r0[1], md.r0[2]}, ap[3] = {md.ap[0], md.ap[1], md.ap[2]};
    const uint8_t mu[3] = {md.mu[0], md.mu[1], md.mu[2]}, om[3] = {md.om[0], md.om[1], md.om[2]},
                  k[3] = {md.k[0], md.k[1], md.k[2]};
    init_chain<1>(c, 0, r0, ap, mu, om, k, b, md.decrypt);
    unsigned long long d[3] = {digest_word(c.x[0]), digest_word(c.y[0]), digest_word(c.z[0])};  // an empty message's
    bool done = seg_run<I, G>(c, w, a.tile, md.in + at, md.out + at, pos, cnt, len, p.state[g], a.dt, a.n_it, lane, d);
    done = done || (valid && len == 0 && round == 0 && lane % G == 0);
    if (done) {
        unsigned long long *t = &a.b.tag_acc[3 * (size_t)i];
        atomicXor(t + 0, d[0]);
        atomicXor(t + 1, d[1]);
        atomicXor(t + 2, d[2]);
    }
}

template <int I, int GA, int GB>
__global__ __launch_bounds__(256) void batch_mix_kernel(BatchArgs a, MixPlan p, uint32_t round) {
    extern __shared__ char lds[];
    mix_round<GA, GB>(
        p, round, *a.b.wide,
        [&](auto g, uint32_t unit, uint32_t first, uint32_t step) __attribute__((always_inline)) {
            batch_mix_body<I, decltype(g)::value>(a, p, round, unit, first, step, lds);
        },
        [&]() __attribute__((always_inline)) { batch_body<1, I, 1>(a, lds); });
}

// One workgroup per message: tag out (encrypt) or tag check, status and zeroing (decrypt).
__global__ void batch_finalize_kernel(BatchDev b, int decrypt) {
    const uint32_t i = blockIdx.x;
    if (i >= b.n_msg) return;
    const MsgDesc &md = b.msgs[i];
    const unsigned long long t[3] = {b.tag_acc[3 * (size_t)i], b.tag_acc[3 * (size_t)i + 1],
                                     b.tag_acc[3 * (size_t)i + 2]};
    if (!decrypt) {
        if (threadIdx.x < LZ_TAG_BYTES) {
            const int q = threadIdx.x;
            md.out[md.n + q] = (uint8_t)(t[q / 8] >> (8 * (q % 8)));
        }
        return;
    }
    const uint8_t *stored = md.in + md.n;
    bool ok = true;
    for (int q = 0; q < LZ_TAG_BYTES; ++q) ok = ok && stored[q] == (uint8_t)(t[q / 8] >> (8 * (q % 8)));
    if (threadIdx.x == 0) (*b.status_ref)[i] = ok ? LZ_OK : LZ_E_INTEGRITY;
    if (!ok)
        for (uint64_t j = threadIdx.x; j < md.n; j += blockDim.x) md.out[j] = 0;
}

// ---- served path: resumable chains ------------------------------------------------------

struct TickArgs {
    TickDev t;
    double dt;
    uint32_t n_it, block_len, tile;
};

// Advances the chains of list entries base, base + 1, ... below end, a wave's worth, by up to tick_bytes bytes.
template <int M, int I, int G>
__device__ __forceinline__ void tick_body(const TickArgs &a, const WaveLds &w, uint64_t base, uint64_t end,
                                          uint32_t tick_bytes) {
    const int lane = threadIdx.x % WAVE;
    Chains<M> c;
    const uint8_t *in[M];
    uint8_t *out[M];
    uint32_t cnt[M], slot[M];
    bool valid[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const uint64_t e = base + (uint64_t)m * WAVE + lane / G;
        valid[m] = e < end;
        slot[m] = valid[m] ? a.t.list[e] : 0u;
        cnt[m] = 0;
        in[m] = nullptr;
        out[m] = nullptr;
        if (!valid[m]) {  // past the end of the list: idle lane, touches no memory
            const double z3[3] = {0.0, 0.0, 0.0};
            const uint8_t u3[3] = {0, 0, 0}, k3[3] = {4, 4, 4};
            init_chain<M>(c, m, z3, z3, u3, u3, k3, 0, 0);
            continue;
        }
        const ChainSlot &s = a.t.slots[slot[m]];
        const MsgDesc &md = a.t.reqs[s.req].m;
        const double ap[3] = {md.ap[0], md.ap[1], md.ap[2]};
        const uint8_t k[3] = {md.k[0], md.k[1], md.k[2]};
        if (s.fresh) {
            const double r0[3] = {md.r0[0], md.r0[1], md.r0[2]};
            const uint8_t mu[3] = {md.mu[0], md.mu[1], md.mu[2]}, om[3] = {md.om[0], md.om[1], md.om[2]};
            init_chain<M>(c, m, r0, ap, mu, om, k, s.blk, md.decrypt);
        } else {
            c.x[m] = s.r[0]; c.y[m] = s.r[1]; c.z[m] = s.r[2];
            c.a0[m] = s.al[0]; c.a1[m] = s.al[1]; c.a2[m] = s.al[2];
            c.mu0[m] = s.mu[0]; c.mu1[m] = s.mu[1]; c.mu2[m] = s.mu[2];
            c.om0[m] = s.om[0]; c.om1[m] = s.om[1]; c.om2[m] = s.om[2];
            c.ap0[m] = ap[0]; c.ap1[m] = ap[1]; c.ap2[m] = ap[2];
            c.k0[m] = k[0]; c.k1[m] = k[1]; c.k2[m] = k[2];
            c.dec[m] = md.decrypt;
        }
        const uint32_t left = s.len - s.pos;
        cnt[m] = left < tick_bytes ? left : tick_bytes;
        const uint64_t off = (uint64_t)s.blk * a.block_len + s.pos;
        in[m] = md.in + off;
        out[m] = md.out + off;
    }
    wave_run<M, I, G>(c, w, (int)a.tile, in, out, cnt, a.dt, a.n_it, lane, [&](int m) __attribute__((always_inline)) {
        if (!valid[m]) return;
        ChainSlot &s = a.t.slots[slot[m]];
        s.r[0] = c.x[m]; s.r[1] = c.y[m]; s.r[2] = c.z[m];
        s.al[0] = c.a0[m]; s.al[1] = c.a1[m]; s.al[2] = c.a2[m];
        s.mu[0] = (uint8_t)c.mu0[m]; s.mu[1] = (uint8_t)c.mu1[m]; s.mu[2] = (uint8_t)c.mu2[m];
        s.om[0] = (uint8_t)c.om0[m]; s.om[1] = (uint8_t)c.om1[m]; s.om[2] = (uint8_t)c.om2[m];
    });
#pragma unroll
    for (int m = 0; m < M; ++m) {
        if (!valid[m] || lane % G != 0) continue;
        ChainSlot &s = a.t.slots[slot[m]];
        s.fresh = 0;
        s.pos += cnt[m];
        if (s.pos != s.len) continue;
        ReqDesc &rq = a.t.reqs[s.req];
        atomicXor(&rq.tag[0], digest_word(s.r[0]));
        atomicXor(&rq.tag[1], digest_word(s.r[1]));
        atomicXor(&rq.tag[2], digest_word(s.r[2]));
        __threadfence();
        if (atomicSub(&rq.remaining, 1u) != 1u) continue;
        // last chain of the request: every other chain's tag XOR is visible
        __threadfence();
        const unsigned long long t[3] = {atomicXor(&rq.tag[0], 0ull), atomicXor(&rq.tag[1], 0ull),
                                         atomicXor(&rq.tag[2], 0ull)};
        int32_t st = LZ_OK;
        if (!rq.m.decrypt) {
            for (int q = 0; q < LZ_TAG_BYTES; ++q) rq.m.out[rq.m.n + q] = (uint8_t)(t[q / 8] >> (8 * (q % 8)));
        } else {
            for (int q = 0; q < LZ_TAG_BYTES; ++q)
                if (rq.stored_tag[q] != (uint8_t)(t[q / 8] >> (8 * (q % 8)))) st = LZ_E_INTEGRITY;
        }
        rq.status = st;
        const uint32_t at = atomicAdd(a.t.done_count, 1u);
        a.t.done_queue[at] = (s.req << 1) | (st != LZ_OK ? 1u : 0u);
    }
}

// Takes a tick's workgroup off the count.  The last to end sees the waves of other work on the device alone: the server
// reads the least of what they see, as ~*others.
__device__ __forceinline__ void tick_done(const TickArgs &a, uint32_t waves) {
    if (threadIdx.x == 0) atomicMax(a.t.others, ~(atomicSub(&g_waves, waves) - waves));
}

// A tick has the device to itself as a rule, so a short one runs wide without a claim (whose launch would be 6 us a tick, 0.6% of
// a burst of 12,000 chains).  Beside a message, whichever started first keeps its SIMDs, so neither loses by the tick's
// width, and two servers of 12,000 chains each take 26 ms with wide ticks and 31 with a lane per chain.
template <int M, int I, int G>
__global__ __launch_bounds__(256) void tick_kernel(TickArgs a) {
    extern __shared__ char lds[];
    constexpr int ROWS = WAVE * M / G;
    const int wid = threadIdx.x / WAVE, wpw = blockDim.x / WAVE;
    count_waves(wpw);
    const WaveLds w = wave_lds<ROWS>(lds + (size_t)wid * wave_lds_bytes(ROWS, a.tile), a.tile);
    tick_body<M, I, G>(a, w, ((uint64_t)blockIdx.x * wpw + wid) * ROWS, a.t.n_list, a.t.tick_bytes);
    tick_done(a, wpw);
}

// A tick between the chain counts of two layouts (see plan_mix): its list's first n_narrow chains run a lane each
// by narrow_bytes, the others in G lanes by tick_bytes, which takes the same time; the server gives the
// wide places to the requests with the most bytes left.  A burst of 88,000 chains, 22,272 of them behind 65,536, ends after
// 41.1 ms instead of 43.3; requests arriving at 0.3, 0.5 and 0.7 of capacity have a median latency of 16.2, 18.6 and
// 20.1 ms, 18.7, 20.4 and 20.6 without mixed ticks.
template <int I, int G>
__global__ __launch_bounds__(256) void tick_mix_kernel(TickArgs a) {
    extern __shared__ char lds[];
    const int wid = threadIdx.x / WAVE, wpw = blockDim.x / WAVE;
    count_waves(wpw);
    char *p = lds + (size_t)wid * wave_lds_bytes(WAVE, a.tile);
    const uint32_t v = __builtin_amdgcn_readfirstlane(blockIdx.x * wpw + wid), narrow = (a.t.n_narrow + WAVE - 1) / WAVE;
    if (v < narrow)
        tick_body<1, I, 1>(a, wave_lds<WAVE>(p, a.tile), (uint64_t)v * WAVE, a.t.n_narrow, a.t.narrow_bytes);
    else
        tick_body<1, I, G>(a, wave_lds<WAVE / G>(p, a.tile), a.t.n_narrow + (uint64_t)(v - narrow) * (WAVE / G), a.t.n_list,
                           a.t.tick_bytes);
    tick_done(a, wpw);
}

// ---- streaming ----------------------------------------------------------------------------

// End of a stream: fold in the pending partial block (or, for an empty message, block 0's
// initial state), then write the tag (encrypt) or compare it (decrypt).
__global__ void stream_finish_kernel(const ChainSlot *slot, int pending, int empty, double r00, double r01, double r02,
                                     unsigned long long *tag_acc, int decrypt, uint8_t *tag, int32_t *status) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    unsigned long long t[3] = {tag_acc[0], tag_acc[1], tag_acc[2]};
    if (pending) {
        t[0] ^= digest_word(slot->r[0]);
        t[1] ^= digest_word(slot->r[1]);
        t[2] ^= digest_word(slot->r[2]);
    } else if (empty) {
        t[0] ^= digest_word(r00);
        t[1] ^= digest_word(r01);
        t[2] ^= digest_word(r02);
    }
    if (!decrypt) {
        for (int q = 0; q < LZ_TAG_BYTES; ++q) tag[q] = (uint8_t)(t[q / 8] >> (8 * (q % 8)));
        return;
    }
    bool ok = true;
    for (int q = 0; q < LZ_TAG_BYTES; ++q) ok = ok && tag[q] == (uint8_t)(t[q / 8] >> (8 * (q % 8)));
    *status = ok ? LZ_OK : LZ_E_INTEGRITY;
}

// ---- the method's scalar pieces over arrays, for checking them one by one -----------

__global__ void unit_r_kernel(const double *alpha, const uint8_t *om, size_t n, uint8_t *out) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        out[i] = (uint8_t)r_nu(alpha[i], om[i] & 3u);
}

__global__ void unit_theta_kernel(const uint8_t *p, const uint8_t *o3, size_t n, double *out) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        out[i] = theta_of(p[i], o3[i] & 3u);
}

// F^steps of Step 2 (the cipher kernels' loop) on each state (x, y, z).
template <int I>
__global__ void unit_lorenz_kernel(double *r, size_t n, double dt, uint32_t steps) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double x[1] = {r[3 * i]}, y[1] = {r[3 * i + 1]}, z[1] = {r[3 * i + 2]};
    lorenz_steps<1, I>(x, y, z, dt, steps);
    r[3 * i] = x[0];
    r[3 * i + 1] = y[0];
    r[3 * i + 2] = z[0];
}

// Zeroes the body of each listed request (failed decryptions), one workgroup each.
__global__ void req_zero_kernel(const ReqDesc *reqs, const uint32_t *ids, uint32_t n) {
    if (blockIdx.x >= n) return;
    const MsgDesc &md = reqs[ids[blockIdx.x]].m;
    for (uint64_t j = threadIdx.x; j < md.n; j += blockDim.x) md.out[j] = 0;
}

// Installs newly admitted requests: record i goes to reqs[meta[3i]], and its
// meta[3i+1] chains (slot indices idx[meta[3i+2] ..]) start fresh at byte 0.
__global__ void install_kernel(ReqDesc *reqs, ChainSlot *slots, const ReqDesc *staged, const uint32_t *meta,
                               const uint32_t *idx, uint32_t n_new, uint32_t block_len) {
    const uint32_t i = blockIdx.x;
    if (i >= n_new) return;
    const uint32_t rs = meta[3 * i], nb = meta[3 * i + 1], first = meta[3 * i + 2];
    if (threadIdx.x == 0) reqs[rs] = staged[i];
    const uint64_t n = staged[i].m.n;
    for (uint32_t b = threadIdx.x; b < nb; b += blockDim.x) {
        ChainSlot &c = slots[idx[first + b]];
        const uint64_t off = (uint64_t)b * block_len;
        c.fresh = 1;
        c.pos = 0;
        c.len = n == 0 ? 0u : (uint32_t)(n - off < block_len ? n - off : block_len);
        c.req = rs;
        c.blk = b;
    }
}

template <int V>
using Int = std::integral_constant<int, V>;

template <int M, typename F>
hipError_t dispatch_i(uint32_t integ, F f) {
    switch (integ) {
        case LZ_INTEGRATOR_EULER: return f(Int<M>{}, Int<0>{}, Int<1>{});
        case LZ_INTEGRATOR_EULER_FMA: return f(Int<M>{}, Int<1>{}, Int<1>{});
        case LZ_INTEGRATOR_RK4: return f(Int<M>{}, Int<2>{}, Int<1>{});
        default: return hipErrorInvalidValue;
    }
}

// The launches with several lanes per chain (lanes_per_chain names no others).
template <typename F>
hipError_t dispatch_wide(int g, uint32_t integ, F f) {
    if (g == 16 && integ == LZ_INTEGRATOR_EULER) return f(Int<1>{}, Int<0>{}, Int<16>{});
    if (g == 16 && integ == LZ_INTEGRATOR_EULER_FMA) return f(Int<1>{}, Int<1>{}, Int<16>{});
    if (g == 16) return f(Int<1>{}, Int<2>{}, Int<16>{});
    if (g == 4 && integ == LZ_INTEGRATOR_EULER) return f(Int<1>{}, Int<0>{}, Int<4>{});
    if (g == 4 && integ == LZ_INTEGRATOR_RK4) return f(Int<1>{}, Int<2>{}, Int<4>{});
    return hipErrorInvalidValue;
}

// Calls f(M, I, G) with the compile-time chains per lane, integrator and lanes per chain of the launch.
template <typename F>
hipError_t dispatch(int m, int g, uint32_t integ, F f) {
    switch (m) {
        case 1: return g == 1 ? dispatch_i<1>(integ, f) : dispatch_wide(g, integ, f);
        case 2: return dispatch_i<2>(integ, f);
        case 4: return dispatch_i<4>(integ, f);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// a wide launch keeps the LDS of one chain per lane: it may have to run that way
size_t lds_bytes(const KernelShape &sh) { return (size_t)(sh.wg / WAVE) * wave_lds_bytes(WAVE * sh.m, sh.tile); }

// Lanes per chain of a launch of `chains` chains with m per lane on `simds` SIMDs: the most that still
// make at most one wave per SIMD of all the chains.  Such a launch takes one chain's serial time, and
// a step takes 40.6 clocks with 16 lanes (8 instructions instead of 9 for the fused Euler map), 44.6 with
// 4 (RK4: 173.5 with 16, 190 with 4 and 262 with one) and 56.6 with one; with a second wave on a SIMD even two waves of 16 lanes'
// 81 clocks would be more than the 56.6 of one chain per lane.  Four lanes gain nothing for the fused Euler map (9
// instructions either way).
// Measured, 16 / 4 / 1 lanes: 64 KiB in 13.2 / 14.5 / 18.3 ms; 3 MB in - / 14.6 / 18.5; 256 KiB of the
// RK4 format in 56.0 / 60.7 / 92.0; 2048 sequential messages in 211 / 230 / 292.
int lanes_per_chain(uint64_t chains, int m, uint32_t integ, int simds) {
    const uint64_t lanes = (uint64_t)simds * WAVE;
    if (m != 1) return 1;
    if (chains * 16 <= lanes) return 16;
    if (integ != LZ_INTEGRATOR_EULER_FMA && chains * 4 <= lanes) return 4;
    return 1;
}

// A launch of W waves on S SIMDs takes ceil(W / S) waves' time, since a wave's chains cannot be cut among
// SIMDs: 24 MB are 1.43 waves per SIMD and took the time of two.  Chains can be cut in time, though.  The
// last P = S + W mod S waves are advanced in rounds of S waves, one wave on every SIMD, each by one
// segment of its chains' bytes, round-robin: wave w's segments are P >= S tasks apart, so no round holds
// two of them and a round finds the checkpoints of the one before.  The P waves then take P / S waves' time
// and a launch per round.  The other waves, a multiple of S, run at once before them.
//
// `lens` gives the longest chain of each of the P waves (descending; NULL: all block_len, but `last` in the last
// wave: a message one block over a full wave may end in a short one, and 16 MiB + 1 byte took 19.8 ms by a plan, 18.7 without).  Waves past
// a short chain's end have no tasks, so off[] counts the waves that have a segment s.  The segment
// count is the one of 4, 8, 16, 32 with the least predicted time, clocks per step as measured (4 per
// instruction) and SEG_ROUND_US for a launch, its checkpoints and the gap before it; without 2% of
// gain (short steps, or W just below a multiple of S) no plan is made.  Measured: 24 MB in 27.1 ms,
// 39.0 without a plan; 512 files of 79 MB in 89.1 and 93.0.  A round of one wave per SIMD takes 1.18 ms
// per 16 bytes, the rate of 64 MiB in one launch: the part's clock under a full load.
SegPlan plan_segments(uint64_t chains, const uint32_t *lens, uint32_t last, const lz_params &prm, int simds) {
    constexpr double SEG_ROUND_US = 10.0, CLOCKS_PER_US = 2400.0;
    SegPlan best{};
    const uint64_t W = (chains + WAVE - 1) / WAVE, S = (uint64_t)simds;
    if (S == 0 || W <= S || W % S == 0) return best;
    const uint32_t P = (uint32_t)(S + W % S);
    const double insts = prm.integrator == LZ_INTEGRATOR_RK4 ? 65 : (prm.integrator == LZ_INTEGRATOR_EULER_FMA ? 9 : 14);
    const double byte_us = insts * 4.0 * prm.n_it / CLOCKS_PER_US;
    const uint64_t B = prm.block_len;  // up to 2^32 - 1: the sequential version
    auto longest = [&](uint32_t w) { return lens ? lens[w] : (w + 1 == P ? last : prm.block_len); };
    // without a plan: S waves of full length, then the longest of the others beside them
    double best_us = 0.98 * byte_us * ((double)B + longest((uint32_t)S));
    for (uint32_t n = 4; n <= SEG_MAX; n *= 2) {
        SegPlan p{};
        p.seg_len = (uint32_t)((B + n - 1) / n);
        p.segs = (uint32_t)((B + p.seg_len - 1) / p.seg_len);
        bool apart = true;
        for (uint32_t s = 0; s < p.segs; ++s) {
            uint32_t k = P;
            while (k > 0 && s > 0 && longest(k - 1) <= (uint64_t)s * p.seg_len) --k;
            apart = apart && k >= S;
            p.off[s + 1] = p.off[s] + k;
        }
        if (!apart) continue;
        p.rounds = (uint32_t)((p.off[p.segs] + S - 1) / S);
        const double us = p.rounds * (p.seg_len * byte_us + SEG_ROUND_US);
        if (us >= best_us) continue;
        best_us = us;
        p.waves = P;
        p.chain0 = (W - P) * WAVE;
        best = p;
    }
    return best;
}

// Clocks of a step with one wave per SIMD, g lanes per chain.
static double step_clocks(uint32_t integ, int g) {
    if (integ == LZ_INTEGRATOR_RK4) return g == 16 ? 173.5 : (g == 4 ? 190 : 262);
    if (integ == LZ_INTEGRATOR_EULER_FMA) return g == 16 ? 32.6 : 36.6;
    return g == 16 ? 40.6 : (g == 4 ? 44.6 : 56.6);
}

// Between the chain counts of two layouts (lanes_per_chain) the wider one does not fit and the narrower one leaves SIMDs
// idle: 8 MB are half a wave per SIMD with a lane per chain.  A mix plan runs in rounds in which every SIMD has a wave:
// of U units (a wave of chains in ga lanes each) A run in ga lanes and the rest in gb, gb / ga waves a unit, A
// the least that makes them at most one wave per SIMD; the units take turns, so all advance alike.  A
// round is la bytes in ga lanes and lb in gb, chosen to take the same time.  The plan with the least predicted time is
// taken (a step's clocks as measured, MIX_ROUND_US for a round's launch, checkpoints and gap), if it beats one
// launch in ga lanes by 3%.  Measured (with and without a plan): 4.1 MiB in
// 15.1 and 18.5 ms, 6 MiB 16.5 and 18.5, 8 MiB 17.6 and 18.7, 1.3 MiB 13.8 and 14.6; RK4 at 1.2 MB 58.0 and 61.2, 5 MiB 70.3 and
// 88.9; the fused map at 1.3 MiB 11.3 and 12.0; batches of 5.2 MiB 16.1 and 18.5, 7.7 MiB 17.7 and 18.6.  From 10 MiB on
// the gain would be under 3%.
MixPlan plan_mix(uint64_t chains, const lz_params &prm, int simds) {
    constexpr double MIX_ROUND_US = 12.0, CLOCKS_PER_US = 2400.0;
    MixPlan best{};
    const int ga = lanes_per_chain(chains, 1, prm.integrator, simds);
    const int gb = prm.integrator == LZ_INTEGRATOR_EULER_FMA ? 16 : 4 * ga;
    if (ga >= gb || gb > 16 || chains * ga > (uint64_t)simds * WAVE) return best;
    MixPlan p{};
    p.ga = ga;
    p.gb = gb;
    p.unit = WAVE / ga;
    p.units = (uint32_t)((chains + p.unit - 1) / p.unit);
    const uint32_t K = gb / ga;
    if (p.units * K <= (uint32_t)simds) return best;  // fits gb lanes (only with a partial unit)
    p.a = (p.units * K - simds + K - 2) / (K - 1);
    if (p.a >= p.units) return best;
    const double ca = step_clocks(prm.integrator, ga), cb = step_clocks(prm.integrator, gb);
    const double step_us = prm.n_it / CLOCKS_PER_US;
    double best_us = 0.97 * prm.block_len * ca * step_us;
    // 6 to 32 bytes of the default block of 256, and as many rounds of a longer one
    const uint32_t unit_bytes = prm.block_len > 256 ? prm.block_len / 256 : 1;
    for (p.la = 6 * unit_bytes; p.la <= 32 * unit_bytes; p.la += unit_bytes) {
        p.lb = (uint32_t)(p.la * ca / cb * 1.004);
        // the units with the most turns in ga lanes are the last to end
        uint32_t r = prm.block_len / p.lb;
        auto reached = [&](uint32_t rr) {
            const uint64_t turns = ((uint64_t)rr * p.a + p.units - 1) / p.units;
            return turns * p.la + (rr - turns) * p.lb >= prm.block_len;
        };
        while (!reached(r)) ++r;
        const double us = r * ((p.la * ca > p.lb * cb ? p.la * ca : p.lb * cb) * step_us + MIX_ROUND_US);
        if (us >= best_us) continue;
        best_us = us;
        best = p;
        best.rounds = r;
    }
    return best;
}

// Rounded up, so that no request gets on more slowly than in a tick of one lane per chain (rounded down the burst above
// took 40.1 ms and the median at 0.7 of capacity 20.7). Four lanes gain nothing for the fused Euler map, and 16 beside
// four too little for a tick.
uint32_t tick_narrow_bytes(const lz_params &prm, uint32_t tick_bytes) {
    if (prm.integrator == LZ_INTEGRATOR_EULER_FMA) return 0;
    const double b = tick_bytes * step_clocks(prm.integrator, TICK_MIX_LANES) / step_clocks(prm.integrator, 1);
    return (uint32_t)b + (b > (uint32_t)b ? 1 : 0);
}

// TICK_US: what a tick costs beside its steps, as the gaps between ticks measure.  Without it short ticks were mixed too, which only
// makes more of them: at 10 steps a byte a burst of 32,700 chains took 19 ticks and 1.48 ms, 16 and 1.31 now.
double tick_mix_gain(const lz_params &prm, uint32_t tick_bytes, uint32_t narrow_bytes, uint64_t n, uint64_t w) {
    constexpr double TICK_US = 15.0, CLOCKS_PER_US = 2400.0;
    const double ca = step_clocks(prm.integrator, 1), cb = step_clocks(prm.integrator, TICK_MIX_LANES);
    const double step_us = prm.n_it / CLOCKS_PER_US;
    const double mixed = (narrow_bytes * ca > tick_bytes * cb ? narrow_bytes * ca : tick_bytes * cb) * step_us + TICK_US;
    const double plain = tick_bytes * ca * step_us + TICK_US;
    return ((double)(n - w) * narrow_bytes + (double)w * tick_bytes) / ((double)tick_bytes * n) * plain / mixed;
}

bool shape_valid(const KernelShape &sh, const DevInfo &dev) {
    if (sh.m != 1 && sh.m != 2 && sh.m != 4) return false;
    if (sh.wg != 64 && sh.wg != 128 && sh.wg != 256) return false;
    if (sh.tile != 16 && sh.tile != 32 && sh.tile != 64 && sh.tile != 128) return false;
    if (sh.wps < 1 || sh.wps > 8) return false;
    return lds_bytes(sh) <= (size_t)dev.lds_per_wg_max;
}

hipError_t launch_fill_u64(unsigned long long *p, size_t n, hipStream_t s) {
    const unsigned blocks = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks ? blocks : 1), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

namespace {

PlainArgs plain_args(const KernelShape &sh, const lz_key &key, const lz_params &prm, int decrypt, const uint8_t *in,
                     uint8_t *out, uint64_t n, uint64_t nb, unsigned long long *tag_acc, uint64_t block_base) {
    PlainArgs a{};
    for (int j = 0; j < 3; ++j) {
        a.ap[j] = key.a_prime[j];
        a.r0[j] = key.r0[j];
        a.mu[j] = key.mu[j];
        a.om[j] = key.omega[j];
        a.k[j] = key.k[j];
    }
    a.decrypt = (uint32_t)decrypt;
    a.dt = prm.dt;
    a.n_it = prm.n_it;
    a.block_len = prm.block_len;
    a.tile = (uint32_t)sh.tile;
    a.in = in;
    a.out = out;
    a.n = n;
    a.nb = nb;
    a.block_base = block_base;
    a.tag_acc = tag_acc;
    a.wide = tag_acc + TAG_WIDE;
    return a;
}

// Workgroups of a launch of `chains` chains.
uint64_t grid_of(const KernelShape &sh, uint64_t chains) {
    const uint64_t per_wg = (uint64_t)sh.wg * sh.m / sh.g;
    return (chains + per_wg - 1) / per_wg;
}

}  // namespace

hipError_t launch_claim(const KernelShape &sh, uint64_t grid, unsigned long long *p, size_t n,
                        unsigned long long *wide, hipStream_t s) {
    const unsigned blocks = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    hipLaunchKernelGGL(claim_kernel, dim3(blocks ? blocks : 1), dim3(256), 0, s, p, n, wide,
                       (uint32_t)(grid * sh.wg / WAVE), (uint32_t)sh.simds);
    return hipGetLastError();
}

// After `refused`, the error of a launch whose waves are counted before it runs (by a claim on the stream, or by the rounds before
// it): takes them off, or they would keep later launches of the process narrow.  wide: if the claim was granted (a mix
// plan's first round has given them back otherwise).
hipError_t give_back(hipError_t refused, const KernelShape &sh, uint64_t grid, hipStream_t s,
                     const unsigned long long *wide = nullptr) {
    hipLaunchKernelGGL(give_back_kernel, dim3(1), dim3(1), 0, s, (uint32_t)(grid * sh.wg / WAVE), wide);
    (void)hipGetLastError();
    return refused;
}

// Workgroups of a round of a segment plan: one wave per SIMD, in whole workgroups, so that round r starts at task
// r * waves.
uint64_t seg_grid(const KernelShape &sh) { return (sh.simds + sh.wg / WAVE - 1) / (sh.wg / WAVE); }

// The rounds of a segment plan, whose waves a claim counts: launch(grid, first) starts one.
template <typename F>
hipError_t seg_rounds(const KernelShape &sh, const SegPlan &p, hipStream_t s, F launch) {
    const uint64_t grid = seg_grid(sh);
    for (uint64_t first = 0; first < p.off[p.segs]; first += grid * (sh.wg / WAVE)) {
        const hipError_t e = launch((unsigned)grid, first);
        if (e != hipSuccess) return give_back(e, sh, grid, s);
    }
    return hipSuccess;
}

// The tile that holds a segment, as far as there is one.
int seg_tile(uint32_t seg_len, int most) {
    int tile = 16;
    while (tile < (int)seg_len && tile < most) tile *= 2;
    return tile;
}

// The rounds of a mix plan, each launched by launch(integrator, lanes, lanes, shape, grid, round); p, n: words to
// clear first (the tags of whole messages).
template <class Launch>
hipError_t mix_rounds(const KernelShape &shape, uint32_t integ, const MixPlan &plan, unsigned long long *p, size_t n,
                      unsigned long long *wide, hipStream_t s, Launch &&launch) {
    KernelShape sh = shape;
    sh.tile = seg_tile(plan.lb, sh.tile);
    const uint32_t waves = plan.a + (plan.units - plan.a) * (plan.gb / plan.ga), wpw = sh.wg / WAVE;
    const unsigned grid = (waves + wpw - 1) / wpw;
    hipError_t e = launch_claim(sh, grid, p, n, wide, s);
    if (e != hipSuccess) return e;
    for (uint32_t r = 0; r < plan.rounds; ++r) {
        auto run = [&](auto ic, auto ac, auto bc) {
            launch(ic, ac, bc, sh, grid, r);
            return hipGetLastError();
        };
        if (integ == LZ_INTEGRATOR_EULER && plan.ga == 1) e = run(Int<0>{}, Int<1>{}, Int<4>{});
        else if (integ == LZ_INTEGRATOR_EULER) e = run(Int<0>{}, Int<4>{}, Int<16>{});
        else if (integ == LZ_INTEGRATOR_EULER_FMA) e = run(Int<1>{}, Int<1>{}, Int<16>{});
        else if (plan.ga == 1) e = run(Int<2>{}, Int<1>{}, Int<4>{});
        else e = run(Int<2>{}, Int<4>{}, Int<16>{});
        if (e != hipSuccess) return give_back(e, sh, grid, s, r == 0 ? nullptr : wide);
    }
    return hipSuccess;
}

template <bool X>
hipError_t launch_mix(const KernelShape &shape, const PlainArgs &args, uint32_t integ, const MixPlan &plan,
                      unsigned long long *p, size_t n, hipStream_t s) {
    return mix_rounds(shape, integ, plan, p, n, args.tag_acc + TAG_WIDE, s,
                      [&](auto ic, auto ac, auto bc, const KernelShape &sh, unsigned grid, uint32_t r) {
        constexpr int I = decltype(ic)::value, GA = decltype(ac)::value, GB = decltype(bc)::value;
        PlainArgs a = args;
        a.tile = (uint32_t)sh.tile;
        hipLaunchKernelGGL((mix_kernel<I, X, GA, GB>), dim3(grid), dim3(sh.wg), lds_bytes(sh), s, a, plan, r);
    });
}

hipError_t launch_plain(const KernelShape &sh, const lz_key &key, const lz_params &prm, int decrypt,
                        const uint8_t *in, uint8_t *out, uint64_t n, unsigned long long *tag_acc, const SegPlan &plan,
                        const MixPlan &mix, hipStream_t s) {
    const uint64_t nb = n == 0 ? 1 : (n + prm.block_len - 1) / prm.block_len;
    PlainArgs a = plain_args(sh, key, prm, decrypt, in, out, n, nb, tag_acc, 0);
    if (mix.rounds) return launch_mix<false>(sh, a, prm.integrator, mix, tag_acc, TAG_WORDS, s);
    if (plan.waves) a.nb = plan.chain0;
    const uint64_t grid = grid_of(sh, a.nb);
    const uint64_t claim = plan.waves ? seg_grid(sh) : (sh.g > 1 ? grid : 0);  // workgroups counted before they run
    hipError_t e = claim ? launch_claim(sh, claim, tag_acc, TAG_WORDS, tag_acc + TAG_WIDE, s)
                         : launch_fill_u64(tag_acc, TAG_WORDS, s);
    if (e != hipSuccess) return e;
    if (grid) {
        e = dispatch(sh.m, sh.g, prm.integrator, [&](auto mc, auto ic, auto gc) {
            constexpr int M = decltype(mc)::value;
            constexpr int I = decltype(ic)::value;
            constexpr int G = decltype(gc)::value;
            hipLaunchKernelGGL((plain_kernel<M, I, false, G>), dim3((unsigned)grid), dim3(sh.wg), lds_bytes(sh), s, a);
            return hipGetLastError();
        });
        if (e != hipSuccess) return claim ? give_back(e, sh, claim, s) : e;
    }
    if (!plan.waves) return hipSuccess;
    KernelShape ss = sh;
    ss.tile = seg_tile(plan.seg_len, sh.tile);
    a.nb = nb;
    a.tile = (uint32_t)ss.tile;
    return seg_rounds(ss, plan, s, [&](unsigned g, uint64_t first) {
        return dispatch_i<1>(prm.integrator, [&](auto, auto ic, auto) {
            constexpr int I = decltype(ic)::value;
            hipLaunchKernelGGL((plain_seg_kernel<I>), dim3(g), dim3(ss.wg), lds_bytes(ss), s, a, plan, first);
            return hipGetLastError();
        });
    });
}

hipError_t launch_stream_step(const KernelShape &shape, const lz_key &key, const lz_params &prm, int decrypt,
                              const uint8_t *in, uint8_t *out, uint64_t full, uint64_t block_base,
                              const StreamExtra &x, unsigned long long *tag_acc, const MixPlan &mix, hipStream_t s) {
    const uint64_t lanes = full + (x.head_slot ? 1 : 0) + (x.tail_slot ? 1 : 0);
    if (lanes == 0) return hipSuccess;
    KernelShape sh{1, shape.wg, shape.tile, shape.wps};
    sh.simds = shape.simds;
    sh.g = lanes_per_chain(lanes, 1, prm.integrator, sh.simds);
    PlainArgs a = plain_args(sh, key, prm, decrypt, in, out, full * prm.block_len, full, tag_acc, block_base);
    a.x = x;
    if (mix.rounds) return launch_mix<true>(sh, a, prm.integrator, mix, nullptr, 0, s);
    const uint64_t grid = grid_of(sh, lanes);
    if (sh.g > 1) {
        const hipError_t e = launch_claim(sh, grid, nullptr, 0, tag_acc + TAG_WIDE, s);
        if (e != hipSuccess) return e;
    }
    const size_t lds = lds_bytes(sh);
    const hipError_t e = dispatch(1, sh.g, prm.integrator, [&](auto, auto ic, auto gc) {
        constexpr int I = decltype(ic)::value;
        constexpr int G = decltype(gc)::value;
        hipLaunchKernelGGL((plain_kernel<1, I, true, G>), dim3((unsigned)grid), dim3(sh.wg), lds, s, a);
        return hipGetLastError();
    });
    return e != hipSuccess && sh.g > 1 ? give_back(e, sh, grid, s) : e;
}

hipError_t launch_plain_finalize(int decrypt, const unsigned long long *tag_acc, const uint8_t *stored_tag,
                                 uint8_t *tag_out, int32_t *status, uint8_t *body, uint64_t n, hipStream_t s) {
    unsigned blocks = 1;
    if (decrypt) {
        const uint64_t want = (n + 256 * 16 - 1) / (256 * 16);
        blocks = (unsigned)(want < 1 ? 1 : (want > 2048 ? 2048 : want));
    }
    hipLaunchKernelGGL(plain_finalize_kernel, dim3(blocks), dim3(256), 0, s, decrypt, tag_acc, stored_tag, tag_out,
                       status, body, n);
    return hipGetLastError();
}

hipError_t launch_batch(const KernelShape &sh, const DevInfo &dev, const lz_params &prm, const BatchDev &b,
                        const SegPlan &plan, const MixPlan &mix, hipStream_t s) {
    BatchArgs a;
    a.b = b;
    a.dt = prm.dt;
    a.n_it = prm.n_it;
    a.block_len = prm.block_len;
    a.tile = (uint32_t)sh.tile;
    a.n_chains = plan.waves ? plan.chain0 : b.n_full + b.n_tail;
    // persistent grid: wps waves on each of the 4 SIMDs of every CU, but no more than the tasks
    const uint64_t waves = (uint64_t)dev.cus * CU_SIMDS * sh.wps;
    const uint64_t wpw = (uint64_t)sh.wg / WAVE;
    uint64_t grid = (waves + wpw - 1) / wpw;
    const uint64_t need = grid_of(sh, a.n_chains);
    if (need < grid) grid = need;
    const size_t words = 3 * (size_t)b.n_msg + 1;  // tags and the work-queue counter
    if (mix.rounds)
        return mix_rounds(sh, prm.integrator, mix, b.tag_acc, words, b.wide, s,
                          [&](auto ic, auto ac, auto bc, const KernelShape &ms, unsigned g, uint32_t r) {
            constexpr int I = decltype(ic)::value, GA = decltype(ac)::value, GB = decltype(bc)::value;
            a.tile = (uint32_t)ms.tile;
            hipLaunchKernelGGL((batch_mix_kernel<I, GA, GB>), dim3(g), dim3(ms.wg), lds_bytes(ms), s, a, mix, r);
        });
    const uint64_t claim = plan.waves ? seg_grid(sh) : (sh.g > 1 ? grid : 0);  // workgroups counted before they run
    hipError_t e = claim ? launch_claim(sh, claim, b.tag_acc, words, b.wide, s)
                         : launch_fill_u64(b.tag_acc, words, s);
    if (e != hipSuccess) return e;
    if (grid) {
        e = dispatch(sh.m, sh.g, prm.integrator, [&](auto mc, auto ic, auto gc) {
            constexpr int M = decltype(mc)::value;
            constexpr int I = decltype(ic)::value;
            constexpr int G = decltype(gc)::value;
            hipLaunchKernelGGL((batch_kernel<M, I, G>), dim3((unsigned)grid), dim3(sh.wg), lds_bytes(sh), s, a);
            return hipGetLastError();
        });
        if (e != hipSuccess) return claim ? give_back(e, sh, claim, s) : e;
    }
    if (!plan.waves) return hipSuccess;
    KernelShape ss = sh;
    ss.tile = seg_tile(plan.seg_len, sh.tile);
    a.tile = (uint32_t)ss.tile;
    return seg_rounds(ss, plan, s, [&](unsigned g, uint64_t first) {
        return dispatch_i<1>(prm.integrator, [&](auto, auto ic, auto) {
            constexpr int I = decltype(ic)::value;
            hipLaunchKernelGGL((batch_seg_kernel<I>), dim3(g), dim3(ss.wg), lds_bytes(ss), s, a, plan, first);
            return hipGetLastError();
        });
    });
}

hipError_t launch_set_status_ref(int32_t **slot, int32_t *status, hipStream_t s) {
    hipLaunchKernelGGL(set_status_ref_kernel, dim3(1), dim3(1), 0, s, slot, status);
    return hipGetLastError();
}

hipError_t launch_batch_finalize(const BatchDev &b, int decrypt, hipStream_t s) {
    hipLaunchKernelGGL(batch_finalize_kernel, dim3(b.n_msg ? b.n_msg : 1), dim3(256), 0, s, b, decrypt);
    return hipGetLastError();
}

hipError_t launch_tick(const KernelShape &sh, const lz_params &prm, const TickDev &t, hipStream_t s) {
    if (t.n_list == 0) return hipSuccess;
    TickArgs a;
    a.t = t;
    a.dt = prm.dt;
    a.n_it = prm.n_it;
    a.block_len = prm.block_len;
    a.tile = (uint32_t)sh.tile;
    const size_t lds = lds_bytes(sh);
    if (t.narrow_bytes) {
        constexpr int G = TICK_MIX_LANES;
        const uint32_t per = WAVE / G, wpw = sh.wg / WAVE;
        const uint32_t waves = (t.n_narrow + WAVE - 1) / WAVE + (t.n_list - t.n_narrow + per - 1) / per;
        const dim3 grid((waves + wpw - 1) / wpw), wg(sh.wg);
        if (prm.integrator == LZ_INTEGRATOR_EULER) hipLaunchKernelGGL((tick_mix_kernel<0, G>), grid, wg, lds, s, a);
        else if (prm.integrator == LZ_INTEGRATOR_RK4) hipLaunchKernelGGL((tick_mix_kernel<2, G>), grid, wg, lds, s, a);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    const uint64_t grid = grid_of(sh, t.n_list);
    return dispatch(sh.m, sh.g, prm.integrator, [&](auto mc, auto ic, auto gc) {
        constexpr int M = decltype(mc)::value;
        constexpr int I = decltype(ic)::value;
        constexpr int G = decltype(gc)::value;
        hipLaunchKernelGGL((tick_kernel<M, I, G>), dim3((unsigned)grid), dim3(sh.wg), lds, s, a);
        return hipGetLastError();
    });
}

hipError_t read_waves(uint32_t *waves, hipStream_t s) {
    const hipError_t e = hipMemcpyFromSymbolAsync(waves, HIP_SYMBOL(g_waves), sizeof *waves, 0, hipMemcpyDeviceToHost, s);
    return e == hipSuccess ? hipStreamSynchronize(s) : e;
}

hipError_t launch_unit_r(const double *alpha, const uint8_t *om, size_t n, uint8_t *out, hipStream_t s) {
    const size_t blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
    hipLaunchKernelGGL(unit_r_kernel, dim3((unsigned)(blocks ? blocks : 1)), dim3(256), 0, s, alpha, om, n, out);
    return hipGetLastError();
}

hipError_t launch_unit_theta(const uint8_t *p, const uint8_t *o3, size_t n, double *out, hipStream_t s) {
    const size_t blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
    hipLaunchKernelGGL(unit_theta_kernel, dim3((unsigned)(blocks ? blocks : 1)), dim3(256), 0, s, p, o3, n, out);
    return hipGetLastError();
}

hipError_t launch_unit_lorenz(const lz_params &prm, double *r, size_t n, uint32_t steps, hipStream_t s) {
    const size_t blocks = (n + 255) / 256;
    return dispatch_i<1>(prm.integrator, [&](auto, auto ic, auto) {
        constexpr int I = decltype(ic)::value;
        hipLaunchKernelGGL((unit_lorenz_kernel<I>), dim3((unsigned)blocks), dim3(256), 0, s, r, n, prm.dt, steps);
        return hipGetLastError();
    });
}

hipError_t launch_stream_finish(const ChainSlot *slot, int pending, int empty, const lz_key &key,
                                unsigned long long *tag_acc, int decrypt, uint8_t *tag, int32_t *status,
                                hipStream_t s) {
    hipLaunchKernelGGL(stream_finish_kernel, dim3(1), dim3(64), 0, s, slot, pending, empty, key.r0[0], key.r0[1],
                       key.r0[2], tag_acc, decrypt, tag, status);
    return hipGetLastError();
}

hipError_t launch_install(ReqDesc *reqs, ChainSlot *slots, const ReqDesc *staged, const uint32_t *meta,
                          const uint32_t *idx, uint32_t n_new, uint32_t block_len, hipStream_t s) {
    if (n_new == 0) return hipSuccess;
    hipLaunchKernelGGL(install_kernel, dim3(n_new), dim3(256), 0, s, reqs, slots, staged, meta, idx, n_new,
                       block_len);
    return hipGetLastError();
}

hipError_t launch_req_zero(const ReqDesc *reqs, const uint32_t *req_ids, uint32_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(req_zero_kernel, dim3(n), dim3(256), 0, s, reqs, req_ids, n);
    return hipGetLastError();
}

}  // namespace lz
