// hp_device.h -- device functions that the stencil kernels share.
#pragma once

#include <hip/hip_runtime.h>

namespace hp {

// Reciprocal: hardware estimate refined by two Newton steps (error within a couple of ulp).
__device__ __forceinline__ double fast_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// the value that lane `lane` of the wave holds
__device__ __forceinline__ double of_lane(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, lane), hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// kappa = 1/rho at the face between cells of face densities ra and rb. FR = 0 (the default): the
// factor 2 / (ra + rb) of the face-velocity update (step (viii)); FR = 1: the mean of the two
// cells' kappa, (1/ra + 1/rb) / 2.
template <int FR, typename T>
__device__ __forceinline__ T face_kappa(T ra, T rb) {
    if constexpr (FR == 1) return T(0.5) * (fast_rcp(ra) + fast_rcp(rb));
    return T(2) * fast_rcp(ra + rb);
}

// the face rule of a launch as the compile-time constant FRV of the statement it runs
#define WITH_FACE_RULE(rule, ...)      \
    do {                               \
        if (rule) {                    \
            constexpr int FRV = 1;     \
            __VA_ARGS__;               \
        } else {                       \
            constexpr int FRV = 0;     \
            __VA_ARGS__;               \
        }                              \
    } while (0)

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Fine taps of coarse index I along one axis for R = P^T / 2 (P: weights 3/4 parent, 1/4 the
// second-nearest coarse cell; mirrored at a Neumann end, wrapped on a periodic axis): always four
// (index, weight) pairs at 2I - 1 .. 2I + 2; missing taps (Neumann ends, an uncoarsened axis) get
// weight 0 and an in-range index, so the restriction is straight-line code with all its loads
// independent. A coarsened axis has at least four fine cells, so a tap wraps at most once and no
// cell is its own second-nearest except at a Neumann end. (As remainders and comparisons of indices
// the taps cost more than the sums: 64^2 -> 32^2 cells in one workgroup 7.0 us against 2.8.)
__device__ __forceinline__ void restrict_taps(int I, int nf, int coarsened, int periodic, int* idx,
                                              float* w) {
    const int nc = nf >> 1;
    const bool lo = !periodic && I == 0, hi = !periodic && I == nc - 1;
    const int first = 2 * I - 1, last = 2 * I + 2;
    idx[0] = !coarsened ? I : first >= 0 ? first : periodic ? first + nf : 2 * I;
    idx[1] = coarsened ? 2 * I : I;
    idx[2] = coarsened ? 2 * I + 1 : I;
    idx[3] = !coarsened ? I : last < nf ? last : periodic ? last - nf : 2 * I;
    w[0] = !coarsened ? 1.0f : lo ? 0.0f : 0.125f;
    w[1] = !coarsened ? 0.0f : lo ? 0.5f : 0.375f;
    w[2] = !coarsened ? 0.0f : hi ? 0.5f : 0.375f;
    w[3] = !coarsened || hi ? 0.0f : 0.125f;
}

// Coarse taps of fine index i along one axis for P.
// Always two (index, weight) pairs: on an axis that is not coarsened the second has weight 0 and
// the first index again, so the prolongation is straight-line code with independent loads.
__device__ __forceinline__ void prolong_taps(int i, int nc, int coarsened, int periodic, int* idx,
                                             float* w) {
    const int parent = i >> 1;
    int other = (i & 1) ? parent + 1 : parent - 1;
    if (other < 0) other = periodic ? nc - 1 : parent;
    if (other >= nc) other = periodic ? 0 : parent;
    idx[0] = coarsened ? parent : i;
    idx[1] = coarsened ? other : i;
    w[0] = coarsened ? 0.75f : 1.0f;
    w[1] = coarsened ? 0.25f : 0.0f;
}

}  // namespace hp
