// kernels_resident.hpp -- small one-atom 2D lattices with a compile-time
// stencil, advanced many steps per launch by one workgroup (PT sites per
// thread: one up to 1024 sites, two up to 2048 in FP32).
//
// The spins and the predictor live in LDS for the whole launch; a thread
// forms the LDS cells of its neighbours once (wrapped along periodic axes, a
// zero cell past open edges), so a step is predictor, barrier, corrector,
// barrier, with no halo to stage or to refresh and no predictor ring.  What
// bounds it: the vector issue of one CU (FP64 most), below the launch, load
// and drain that a step costs on the tile kernels at these sizes (us per
// step, tile kernel against this one, same bits): square 32^2 FP64 6.9 / 3.5,
// FP32 4.1 / 1.4; triangular 32^2 at 10 K FP64 13.3 / 9.4, FP32 5.3 / 2.5.
#pragma once

#include "kernels_fused2d.hpp"

namespace sp {

// Sites the path takes in an engine precision.
template <typename T>
constexpr int resident_sites() {
    return sizeof(T) == 4 ? 2048 : 1024;
}

// n_steps steps of the solver from n to nout (which may be the same array);
// the Philox step of the first is the one in A_arg's key.
template <typename T, int S, int NDMI, int SOLVER, int PT>
__global__ void __launch_bounds__(1024)
    k_resident2d(StepCoef<T> C, Site2D<T> Q, LLGArgs<T> A_arg, const int* __restrict__ abort_flag, const T* n, T* nout,
                 int n_steps) {
    if (abort_flag && *abort_flag) return;
    using SH = ShapeTab<S>;
    constexpr int CELLS = 1024 * PT;
    __shared__ V4<T> sN[CELLS + 1];
    __shared__ V4<T> sP[CELLS + 1];
    LLGArgs<T> A = A_arg;
    const unsigned long long step0 = ((unsigned long long)A.key.step_hi << 32) | A.key.step_lo;
    const int N = Q.na * Q.nb;
    int site[PT];
    bool own[PT];
    V3<T> ni[PT], base[PT], keep[PT], p[PT];
    int nb[PT][SH::NB];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        site[j] = threadIdx.x + j * blockDim.x;
        own[j] = site[j] < N;
        const int ic = own[j] ? site[j] : N - 1;
        const int y = ic / Q.na, x = ic - y * Q.na;
        ni[j] = load3(n, N, ic);
#pragma unroll
        for (int q = 0; q < SH::NB; ++q) {
            bool in = true;
            const int gx = wrap_once(x + SH::da[q], Q.na, Q.per_a, in);
            const int gy = wrap_once(y + SH::db[q], Q.nb, Q.per_b, in);
            nb[j][q] = in ? gx + gy * Q.na : CELLS;
        }
        if (own[j]) sN[site[j]] = V4<T>{ni[j].x, ni[j].y, ni[j].z, T(0)};
    }
    if (threadIdx.x == 0) sN[CELLS] = sP[CELLS] = V4<T>{T(0), T(0), T(0), T(0)};
    __syncthreads();
    const V3<T> Bext{C.Bext[0], C.Bext[1], C.Bext[2]};
    const T h = rot_half_factor(A.gp, A.dt);
    for (int k = 0; k < n_steps; ++k) {
        const unsigned long long step = step0 + (unsigned long long)k;
        A.key.step_lo = (uint32_t)step;
        A.key.step_hi = (uint32_t)(step >> 32);
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            base[j] = Bext;
            if (A.thermal) {
                asm volatile("");   // the draw stays behind the branch (else it ran at T = 0 too)
                base[j] = base[j] + Q.sigma * normals3(thermal_bits(A.key, (uint32_t)site[j]), T(0));
            }
            const V3<T> B = shape_B_cells<T, S, NDMI>(C, Q, sN, nb[j], ni[j], base[j]);
            if constexpr (SOLVER == SOLVER_HEUN) {
                keep[j] = cross(ni[j], llg_A(ni[j], B, A.gp, A.alpha));
                p[j] = normalize3(ni[j] + A.dt * keep[j]);
            } else if constexpr (SOLVER == SOLVER_SIB) {
                p[j] = T(0.5) * (ni[j] + sib_stage(ni[j], llg_A(ni[j], B, A.gp, A.alpha), A.dt));
            } else {
                keep[j] = llg_w(ni[j], B, A.alpha);
                p[j] = rotate_half(ni[j], keep[j], h);
            }
            if (own[j]) sP[site[j]] = V4<T>{p[j].x, p[j].y, p[j].z, T(0)};
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const V3<T> Bp = shape_B_cells<T, S, NDMI>(C, Q, sP, nb[j], p[j], base[j]);
            if constexpr (SOLVER == SOLVER_HEUN)
                ni[j] = normalize3(ni[j] + (T(0.5) * A.dt) * (keep[j] + cross(p[j], llg_A(p[j], Bp, A.gp, A.alpha))));
            else if constexpr (SOLVER == SOLVER_SIB)
                ni[j] = renorm_if_float(sib_stage(ni[j], llg_A(p[j], Bp, A.gp, A.alpha), A.dt));
            else
                ni[j] = renorm_if_float(rotate_half(ni[j], keep[j] + llg_w(p[j], Bp, A.alpha), T(0.5) * h));
            if (own[j]) sN[site[j]] = V4<T>{ni[j].x, ni[j].y, ni[j].z, T(0)};
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < PT; ++j)
        if (own[j]) store3(nout, N, site[j], ni[j]);
}

}  // namespace sp
