// kernels_resident.hpp -- small one-atom 2D lattices with a compile-time
// stencil, advanced many steps per launch by one workgroup (PT sites per
// thread: one up to 1024 sites, two up to 2048 in FP32).  A launch of a single
// step is shared out over workgroups of a site per thread, which correct
// kResidentSpan sites each and predict those within the stencil's reach of
// them too.
//
// The spins and the predictor live in LDS for the whole launch; a thread
// forms the LDS cells of its neighbours once (wrapped along periodic axes, a
// zero cell past open edges), so a step is predictor, barrier, corrector,
// barrier, with no halo to stage or to refresh and no predictor ring.  What
// bounds it: the vector issue of one CU (FP64 most), below the launch, load
// and drain that a step costs on the tile kernels at these sizes (us per
// step of a run of 100, tile kernel against this one; the same expressions,
// equal to rounding): square 32^2 FP64 6.9 / 3.5, FP32 4.1 / 1.4; triangular
// 32^2 at 10 K FP64 13.3 / 9.4, FP32 5.3 / 2.5; at the upper end, FP32 64 x 32
// with one shell 4.7 / 3.0, with three 5.6 / 4.2 (18 cells read from LDS per
// site and stage bind); observed every step, three shells, 26.4 / 24.7.  A
// launch of a single step there: tile kernel 5.3, one workgroup for all sites
// 8.1, shared out 5.2 (one shell 4.4 against 5.7).
#pragma once

#include "kernels_fused2d.hpp"

namespace sp {

// Sites the path takes in an engine precision.
template <typename T>
constexpr int resident_sites() {
    return sizeof(T) == 4 ? 2048 : 1024;
}

constexpr int kResidentSpan = 128;   // sites a workgroup corrects in a shared launch

// Threads of a shared launch: the sites of the span and those within reach of
// them, less than R + 1 rows away (a neighbour along a row is less than a row
// away, around the end of the lattice too).
__host__ __device__ __forceinline__ int resident_window(int R, int na, int N) {
    const int w = kResidentSpan + 2 * (R + 1) * na;
    return w < N ? w : N;
}

// Neighbour coordinate t, at most one lattice length outside a periodic axis
// (whose length exceeds twice the stencil's reach): two selects.
__device__ __forceinline__ int wrap_near(int t, int n, int per, bool& in) {
    const int w = t < 0 ? t + n : (t >= n ? t - n : t);
    in = in && (per != 0 || w == t);
    return w;
}

// n_steps steps of the solver from n to nout; the Philox step of the first is
// the one in A_arg's key.  One workgroup (nout = n allowed), or several, a
// shared launch of one step with nout apart from n.
template <typename T, int S, int NDMI, int SOLVER, int PT>
__global__ void __launch_bounds__(1024)
    k_resident2d(StepCoef<T> C, Site2D<T> Q, LLGArgs<T> A_arg, const int* __restrict__ abort_flag, const T* n, T* nout,
                 int n_steps) {
    const int stop = abort_flag ? *abort_flag : 0;   // on its way with the spins
    using SH = ShapeTab<S>;
    constexpr int CELLS = 1024 * PT;
    __shared__ V4<T> sN[CELLS + 1];
    __shared__ V4<T> sP[CELLS + 1];
    LLGArgs<T> A = A_arg;
    const unsigned long long step0 = ((unsigned long long)A.key.step_hi << 32) | A.key.step_lo;
    const int N = Q.na * Q.nb;
    const bool shared = gridDim.x > 1;
    const int lo = (int)blockIdx.x * kResidentSpan, window = shared ? resident_window(SH::R, Q.na, N) : N;
    int site[PT];
    bool own[PT], correct[PT];
    V3<T> ni[PT], base[PT], keep[PT], p[PT];
    int nb[PT][SH::NB];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        site[j] = threadIdx.x + j * blockDim.x;
        own[j] = correct[j] = site[j] < window;
        if (shared) {
            if (j > 0) continue;
            int s = lo - (SH::R + 1) * Q.na + (int)threadIdx.x;
            s += s < 0 ? N : 0;
            s -= s >= N ? N : 0;
            site[j] = window < N ? s : (int)threadIdx.x;
            correct[j] = own[j] && site[j] >= lo && site[j] < lo + kResidentSpan;
        }
        const int ic = own[j] ? site[j] : N - 1;
        const int y = ic / Q.na, x = ic - y * Q.na;
        ni[j] = load3(n, N, ic);
#pragma unroll
        for (int q = 0; q < SH::NB; ++q) {
            bool in = true;
            const int gx = wrap_near(x + SH::da[q], Q.na, Q.per_a, in);
            const int gy = wrap_near(y + SH::db[q], Q.nb, Q.per_b, in);
            nb[j][q] = in ? gx + gy * Q.na : CELLS;
        }
        if (own[j]) sN[site[j]] = V4<T>{ni[j].x, ni[j].y, ni[j].z, T(0)};
    }
    if (shared) {   // the neighbours on either side of the window
        const int reach = (SH::R + 1) * Q.na, beyond = min(2 * reach, N - window);
        for (int t = threadIdx.x; t < beyond; t += blockDim.x) {
            int s = lo - 2 * reach + t + (t >= reach || beyond < 2 * reach ? window : 0);
            if (beyond < 2 * reach) s += reach;     // all the rest, from the window's end on
            s += s < 0 ? N : 0;
            s -= s >= N ? N : 0;
            const V3<T> v = load3(n, N, s);
            sN[s] = V4<T>{v.x, v.y, v.z, T(0)};
        }
    }
    if (stop) return;
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
            if (j > 0 && shared) continue;
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
            if (j > 0 && shared) continue;
            if (!correct[j]) continue;
            const V3<T> Bp = shape_B_cells<T, S, NDMI>(C, Q, sP, nb[j], p[j], base[j]);
            if constexpr (SOLVER == SOLVER_HEUN)
                ni[j] = normalize3(ni[j] + (T(0.5) * A.dt) * (keep[j] + cross(p[j], llg_A(p[j], Bp, A.gp, A.alpha))));
            else if constexpr (SOLVER == SOLVER_SIB)
                ni[j] = renorm_if_float(sib_stage(ni[j], llg_A(p[j], Bp, A.gp, A.alpha), A.dt));
            else
                ni[j] = renorm_if_float(rotate_half(ni[j], keep[j] + llg_w(p[j], Bp, A.alpha), T(0.5) * h));
            sN[site[j]] = V4<T>{ni[j].x, ni[j].y, ni[j].z, T(0)};
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < PT; ++j)
        if (correct[j] && !(j > 0 && shared)) store3(nout, N, site[j], ni[j]);
}

}  // namespace sp
