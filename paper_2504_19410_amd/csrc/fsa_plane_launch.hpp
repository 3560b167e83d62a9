// fsa_plane_launch.hpp -- length dispatch of the small-plane launch.  Included by
// one translation unit per precision.
#pragma once

#include "fsa_internal.hpp"
#include "fsa_launch.hpp"
#include "fsa_plane.hpp"

namespace fsa {

// padded lengths of axes 1 and 0 it is compiled for, where the plane fits
#define FSA_PLANE_P_LIST(X, P1) \
    X(P1, 16) X(P1, 24) X(P1, 32) X(P1, 48) X(P1, 64) X(P1, 96) X(P1, 128) X(P1, 192) X(P1, 256)
#define FSA_PLANE_ROWS(X) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(192) X(256)

template <typename R, int P1, int P0>
hipError_t go_plane(const JobPlane& jb, const void* tw1, const void* tw0, hipStream_t st) {
    if constexpr (!Plane<R, P1, P0>::FITS)
        return hipErrorInvalidValue;
    else
        return launch_kernel(k_plane<R, P1, P0>, dim3(jb.H), dim3(Plane<R, P1, P0>::THREADS), 0, st,
                             jb, (const cpx<R>*)tw1, (const cpx<R>*)tw0);
}

template <typename R>
hipError_t PlaneV<R>::launch(int P1, int P0, const JobPlane& jb, const void* tw1, const void* tw0,
                             hipStream_t st) {
    switch (P1 * 4096 + P0) {
#define FSA_CASE(p1, p0) \
    case p1 * 4096 + p0: return go_plane<R, p1, p0>(jb, tw1, tw0, st);
#define FSA_ROW(p1) FSA_PLANE_P_LIST(FSA_CASE, p1)
        FSA_PLANE_ROWS(FSA_ROW)
#undef FSA_ROW
#undef FSA_CASE
    }
    return hipErrorInvalidValue;
}

template <typename R>
bool PlaneV<R>::fits(int P1, int P0) {
    switch (P1 * 4096 + P0) {
#define FSA_CASE(p1, p0) \
    case p1 * 4096 + p0: return Plane<R, p1, p0>::FITS;
#define FSA_ROW(p1) FSA_PLANE_P_LIST(FSA_CASE, p1)
        FSA_PLANE_ROWS(FSA_ROW)
#undef FSA_ROW
#undef FSA_CASE
    }
    return false;
}

template <typename R>
bool PlaneV<R>::faster(int P1, int P0, int H) {
    switch (P1 * 4096 + P0) {
#define FSA_CASE(p1, p0) \
    case p1 * 4096 + p0: \
        return Plane<R, p1, p0>::FITS && \
               !(Plane<R, p1, p0>::FEW_SLOW && H < Plane<R, p1, p0>::FEW);
#define FSA_ROW(p1) FSA_PLANE_P_LIST(FSA_CASE, p1)
        FSA_PLANE_ROWS(FSA_ROW)
#undef FSA_ROW
#undef FSA_CASE
    }
    return false;
}

}  // namespace fsa
