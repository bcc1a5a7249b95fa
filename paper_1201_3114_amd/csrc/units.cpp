// The method's scalar pieces as entry points of their own: R (Eq. R_nu), Theta
// (Step 2) and the iterated map F (Section 3.1, Step 2), each evaluated by the
// same device code as the cipher kernels, so that each can be checked on its
// own against a reference; and what the launches decide by (the plans, the waves in
// flight).
#include <hip/hip_runtime.h>

#include "internal.h"

using namespace lz;

extern "C" int lz_unit_r(lz_ctx *c, const double *d_alpha, const uint8_t *d_omega, size_t n, uint8_t *d_out,
                         void *stream) {
    if (!c || (n && (!d_alpha || !d_omega || !d_out))) return fail(LZ_E_INVAL, "NULL argument");
    if (n == 0) return LZ_OK;
    LZ_HIP(hipSetDevice(c->device));
    LZ_HIP(launch_unit_r(d_alpha, d_omega, n, d_out, (hipStream_t)stream));
    return LZ_OK;
}

extern "C" int lz_unit_theta(lz_ctx *c, const uint8_t *d_p, const uint8_t *d_omega3, size_t n, double *d_out,
                             void *stream) {
    if (!c || (n && (!d_p || !d_omega3 || !d_out))) return fail(LZ_E_INVAL, "NULL argument");
    if (n == 0) return LZ_OK;
    LZ_HIP(hipSetDevice(c->device));
    LZ_HIP(launch_unit_theta(d_p, d_omega3, n, d_out, (hipStream_t)stream));
    return LZ_OK;
}

extern "C" int lz_unit_lorenz(lz_ctx *c, double *d_r, size_t n, uint32_t steps, void *stream) {
    if (!c || (n && !d_r)) return fail(LZ_E_INVAL, "NULL argument");
    if (n > ((size_t)1 << 31)) return fail(LZ_E_INVAL, "at most 2^31 states per call");
    if (n == 0) return LZ_OK;
    LZ_HIP(hipSetDevice(c->device));
    LZ_HIP(launch_unit_lorenz(c->prm, d_r, n, steps, (hipStream_t)stream));
    return LZ_OK;
}

extern "C" int lz_unit_waves(lz_ctx *c, uint32_t *waves, void *stream) {
    if (!c || !waves) return fail(LZ_E_INVAL, "NULL argument");
    LZ_HIP(hipSetDevice(c->device));
    LZ_HIP(read_waves(waves, (hipStream_t)stream));
    return LZ_OK;
}

extern "C" int lz_unit_plan(const lz_params *prm, uint32_t simds, uint64_t chains, const uint32_t *lens,
                            lz_launch_plan *out) {
    if (!prm || !out) return fail(LZ_E_INVAL, "NULL argument");
    if (int rc = lz_params_check(prm)) return rc;
    if (simds == 0 || simds > 65536 || chains == 0 || chains > ((uint64_t)1 << 40)) return fail(LZ_E_INVAL, "no such launch");
    *out = lz_launch_plan{};
    out->lanes = (uint32_t)lanes_per_chain(chains, 1, prm->integrator, (int)simds);
    if (out->lanes == 1) {
        const SegPlan s = plan_segments(chains, lens, prm->block_len, *prm, (int)simds);
        if (s.waves) {
            out->seg_waves = s.waves;
            out->seg_rounds = s.rounds;
            out->segs = s.segs;
            out->seg_len = s.seg_len;
            for (uint32_t i = 0; i <= s.segs; ++i) out->seg_off[i] = s.off[i];
        }
    }
    const MixPlan m = plan_mix(chains, *prm, (int)simds);
    if (m.rounds) {
        out->mix_rounds = m.rounds;
        out->mix_lanes[0] = (uint32_t)m.ga;
        out->mix_lanes[1] = (uint32_t)m.gb;
        out->mix_unit = m.unit;
        out->mix_units = m.units;
        out->mix_first = m.a;
        out->mix_bytes[0] = m.la;
        out->mix_bytes[1] = m.lb;
    }
    return LZ_OK;
}
