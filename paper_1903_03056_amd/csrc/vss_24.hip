// Gain-kernel geometries compiled for N = 24 with a VSS kernel (sigma-dependent kernel
// mode): the same tiles as the VHS family, each direction transformed as one
// complex field (the packed two-field form is not used here).
#include "dealias.hpp"

namespace dgfs {

hipError_t run_vss_24(const dgfs_plan& p, const void* f, void* Q, int nb, Scratch ws, bool pairs, hipStream_t st,
                      hipEvent_t* ev) {
    const int key = p.geo.CH * 100 + p.geo.CZ;
    if (p.precision == DGFS_FP64) {
        switch (key) {
            case 302: return detail::run_slice<double, 24, 3, 2, PIPE_OFF, false, true>(
                p, static_cast<const double*>(f), static_cast<double*>(Q), nb, ws, pairs, st, ev);
            default: return hipErrorInvalidValue;
        }
    }
    switch (key) {
        case 301: return detail::run_slice<float, 24, 3, 1, PIPE_OFF, false, true>(
            p, static_cast<const float*>(f), static_cast<float*>(Q), nb, ws, pairs, st, ev);
        case 302: return detail::run_slice<float, 24, 3, 2, PIPE_OFF, false, true>(
            p, static_cast<const float*>(f), static_cast<float*>(Q), nb, ws, pairs, st, ev);
        case 304: return detail::run_slice<float, 24, 3, 4, PIPE_OFF, false, true>(
            p, static_cast<const float*>(f), static_cast<float*>(Q), nb, ws, pairs, st, ev);
        default: return hipErrorInvalidValue;
    }
}

// The dealiased form on the N = 16 grid, its gain on this NI = 24 grid (the inner
// plan's tile geometry).
hipError_t run_dealias_16(const dgfs_plan& outer, const dgfs_plan& inner, const void* f, void* Q, int nb, void* ws,
                          bool pairs, hipStream_t st, hipEvent_t* ev) {
    const int key = inner.geo.CH * 100 + inner.geo.CZ;
    if (outer.precision == DGFS_FP64) {
        switch (key) {
            case 302: return detail::run_dealiased<double, 16, 3, 2>(
                outer, inner, static_cast<const double*>(f), static_cast<double*>(Q), nb, ws, pairs, st, ev);
            default: return hipErrorInvalidValue;
        }
    }
    switch (key) {
            case 301: return detail::run_dealiased<float, 16, 3, 1>(
                outer, inner, static_cast<const float*>(f), static_cast<float*>(Q), nb, ws, pairs, st, ev);
            case 302: return detail::run_dealiased<float, 16, 3, 2>(
                outer, inner, static_cast<const float*>(f), static_cast<float*>(Q), nb, ws, pairs, st, ev);
            case 304: return detail::run_dealiased<float, 16, 3, 4>(
                outer, inner, static_cast<const float*>(f), static_cast<float*>(Q), nb, ws, pairs, st, ev);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace dgfs
