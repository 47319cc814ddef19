// kernels_pairs.hpp -- tiles of the general path: field, step stages and
// observables of any lattice and bond table (Sec. III.A: pairs of any
// number, range and direction) whose tile and halo fit into LDS.
//
// A workgroup owns a tile of 256 cells (all atoms of the basis) and stages
// its spins with a halo of the table's reach as 16-byte (FP64: 32-byte) LDS
// cells, wrapped along periodic axes and zero outside open ones, so a bond
// is one uniform cell offset: read the cell, multiply, add.  The exchange
// couplings and the DMI vectors are separate lists of (offset, coupling)
// records, staged in LDS too and read as broadcasts (through the scalar cache
// every 64 bytes of a cold list were a miss of their own, 11 of 21 us), so a
// bond without DMI costs three multiply-adds.  The sums run in the order of
// the bond table.
//
// What bounds it: LDS reads, 16 bytes per bond and site.  The site loop it
// replaces on these lattices (k_predict, k_correct, k_gradient,
// k_observe_partial: three wrapped coordinates, six coupling values and three
// loads from memory per bond and site) took 63 us per stage on 48^3 sites
// with 122 bonds, the tiles take 20; it stays for tables whose frame does not
// fit.
#pragma once

#include "kernels_fused2d.hpp"
#include "kernels_reduce.hpp"

namespace sp {

constexpr int kPairCells = 256;      // cells of a tile, one thread each

struct PairTile {
    int log_tx, log_ty, log_tz;      // tile sides (powers of two, 256 cells)
    int W, H, PN;                    // frame: row, rows of a plane, cells per atom
    uint32_t magic_PN, magic_WH, magic_W;   // ceil(2^32 / x): quotients of frame indices
    int ra, rb, rc;                  // halo
    int nx, ny, nz;                  // tiles along a, b, c
};

template <typename T>
struct PairJ {
    int off;
    T J;
};
template <typename T>
struct PairD {
    int off;
    T x, y, z;
};

template <typename T>
struct PairLists {
    const PairJ<T>* j;               // lists of each atom padded to multiples of eight
    const PairD<T>* d;               // and of four (zero couplings, own cell)
    int js[kMaxBasis + 1], ds[kMaxBasis + 1];
};

enum PairStage { PAIR_GRADIENT = 0, PAIR_PREDICT = 1, PAIR_CORRECT = 2, PAIR_OBSERVE = 3 };

// wrap_coord with the usual case, at most one lattice length away, as two
// selects (the division only for frames wider than the lattice).
__device__ __forceinline__ int frame_coord(int t, int n, int per, bool& ok) {
    if (per) {
        t += t < 0 ? n : 0;
        t -= t >= n ? n : 0;
    }
    if (t >= 0 && t < n) return t;
    return wrap_coord(t, n, per, ok);
}

// The field sums of the exchange and DMI lists of one site.
template <typename T>
__device__ __forceinline__ void pair_sums(const PairLists<T>& S, const PairJ<T>* sj, const PairD<T>* sd, int beta,
                                          const V4<T>* cells, int c, V3<T>& gj, V3<T>& gd) {
    gj = gd = V3<T>{T(0), T(0), T(0)};
    const int j1 = S.js[beta + 1];
    for (int q = S.js[beta]; q < j1; q += 8) {
        V3<T> v[8];
        T J[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const PairJ<T> r = sj[q + u];
            J[u] = r.J;
            v[u] = lds_cell_xyz(cells, c + r.off);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) gj = gj - J[u] * v[u];
    }
    const int d1 = S.ds[beta + 1];
    for (int q = S.ds[beta]; q < d1; q += 4) {
        V3<T> v[4], D[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const PairD<T> r = sd[q + u];
            D[u] = V3<T>{r.x, r.y, r.z};
            v[u] = lds_cell_xyz(cells, c + r.off);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) gd = gd - cross(v[u], D[u]);
    }
}

// m: the spins whose field is taken (n, or the predictor's); n, Abuf: start
// of the step and what the predictor kept; out: gradient, predictor or new
// spins; partials: one row of observables per workgroup, which walks the
// tiles with the grid's stride (PAIR_OBSERVE; one tile otherwise).
template <typename T, int STAGE>
__global__ void __launch_bounds__(kPairCells)
    k_pair_tile(Lattice L, PairTile t, PairLists<T> S, Phys<T> P, LLGArgs<T> A_arg, int solver,
                const int* __restrict__ abort_flag, const T* __restrict__ m, const T* __restrict__ n,
                const T* __restrict__ gdd, T* __restrict__ Abuf, T* __restrict__ out, double* __restrict__ partials,
                int tiles) {
    if ((STAGE == PAIR_PREDICT || STAGE == PAIR_CORRECT) && abort_flag && *abort_flag) return;
    extern __shared__ __align__(32) unsigned char pair_smem[];
    V4<T>* cells = reinterpret_cast<V4<T>*>(pair_smem);
    PairJ<T>* sj = reinterpret_cast<PairJ<T>*>(cells + t.PN * L.nb);
    PairD<T>* sd = reinterpret_cast<PairD<T>*>(sj + S.js[L.nb]);
    for (int u = threadIdx.x; u < S.js[L.nb]; u += kPairCells) sj[u] = S.j[u];
    for (int u = threadIdx.x; u < S.ds[L.nb]; u += kPairCells) sd[u] = S.d[u];
    LLGArgs<T> A = A_arg;
    if constexpr (STAGE == PAIR_PREDICT || STAGE == PAIR_CORRECT) A = resolve_step(A_arg);
    const int tid = threadIdx.x;
    const int na = L.n[0], nb = L.n[1], nc = L.n[2], N = L.N;
    const int lx = tid & ((1 << t.log_tx) - 1), ly = (tid >> t.log_tx) & ((1 << t.log_ty) - 1),
              lz = tid >> (t.log_tx + t.log_ty);
    double acc[OBS_NVALS];
    if constexpr (STAGE == PAIR_OBSERVE) {
#pragma unroll
        for (int k = 0; k < OBS_NVALS; ++k) acc[k] = 0.0;
    }
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int bx = tile % t.nx, by = (tile / t.nx) % t.ny, bz = tile / (t.nx * t.ny);
        const int x0 = bx << t.log_tx, y0 = by << t.log_ty, z0 = bz << t.log_tz;
        if (STAGE == PAIR_OBSERVE && tile != (int)blockIdx.x) __syncthreads();   // the last tile is no longer read
        // stage the frame, four cells per thread in flight
        const int staged = t.PN * L.nb;
        for (int u0 = tid; u0 < staged; u0 += 4 * kPairCells) {
            V4<T> v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int u = u0 + k * kPairCells;
                v[k] = V4<T>{T(0), T(0), T(0), T(0)};
                if (u < staged) {
                    const int beta = (int)__umulhi((uint32_t)u, t.magic_PN), r = u - beta * t.PN;
                    const int fz = (int)__umulhi((uint32_t)r, t.magic_WH), rr = r - fz * t.W * t.H;
                    const int fy = (int)__umulhi((uint32_t)rr, t.magic_W), fx = rr - fy * t.W;
                    bool ok = true;
                    const int gx = frame_coord(x0 - t.ra + fx, na, L.per[0], ok);
                    const int gy = frame_coord(y0 - t.rb + fy, nb, L.per[1], ok);
                    const int gz = frame_coord(z0 - t.rc + fz, nc, L.per[2], ok);
                    if (ok) {
                        const V3<T> s = load3(m, N, gx + na * (gy + nb * (gz + nc * beta)));
                        v[k] = V4<T>{s.x, s.y, s.z, T(0)};
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (u0 + k * kPairCells < staged) cells[u0 + k * kPairCells] = v[k];
        }
        __syncthreads();
        const int gx = x0 + lx, gy = y0 + ly, gz = z0 + lz;
        if (gx < na && gy < nb && gz < nc) {
            const int c0 = (lx + t.ra) + t.W * ((ly + t.rb) + t.H * (lz + t.rc));
            for (int beta = 0; beta < L.nb; ++beta) {
                const int i = gx + na * (gy + nb * (gz + nc * beta));
                const int c = c0 + beta * t.PN;
                const V3<T> mi = lds_cell_xyz(cells, c);
                FieldTerms<T> f;
                f.z = V3<T>{P.gZ[beta][0], P.gZ[beta][1], P.gZ[beta][2]};
                const V3<T> ax{P.Kax[beta][0], P.Kax[beta][1], P.Kax[beta][2]};
                f.k = (-P.K2[beta] * dot(ax, mi)) * ax;
                f.q = gauss_gradient(P, mi);
                pair_sums(S, sj, sd, beta, cells, c, f.j, f.d);
                V3<T> g = total(f);
                V3<T> gd{T(0), T(0), T(0)};
                if (gdd) {
                    gd = load3(gdd, N, i);
                    g = g + gd;
                }
                if constexpr (STAGE == PAIR_GRADIENT) {
                    store3(out, N, i, g);
                } else if constexpr (STAGE == PAIR_OBSERVE) {
                    const double sx = mi.x, sy = mi.y, sz = mi.z;
                    if (gdd) acc[OBS_EDD] += 0.5 * (sx * gd.x + sy * gd.y + sz * gd.z);
                    acc[OBS_EZ] += sx * f.z.x + sy * f.z.y + sz * f.z.z;
                    acc[OBS_EK] += 0.5 * (sx * f.k.x + sy * f.k.y + sz * f.k.z) + gauss_energy(P, mi);
                    acc[OBS_EJ] += 0.5 * (sx * f.j.x + sy * f.j.y + sz * f.j.z);
                    acc[OBS_ED] += 0.5 * (sx * f.d.x + sy * f.d.y + sz * f.d.z);
                    const double tx = sy * g.z - sz * g.y, ty = sz * g.x - sx * g.z, tz = sx * g.y - sy * g.x;
                    const double t2 = tx * tx + ty * ty + tz * tz;
                    if (!isfinite(t2)) {
                        acc[OBS_NONFINITE] += 1.0;
                    } else {
                        acc[OBS_TMAX] = fmax(acc[OBS_TMAX], sqrt(t2));
                        acc[OBS_T2] += t2;
                    }
                    acc[OBS_MX] += sx;
                    acc[OBS_MY] += sy;
                    acc[OBS_MZ] += sz;
                    acc[OBS_NDEV] = fmax(acc[OBS_NDEV], fabs(sqrt(sx * sx + sy * sy + sz * sz) - 1.0));
                } else {
                    const T inv_m = T(1) / P.mumuB[beta];
                    V3<T> B = (-inv_m) * g;
                    if (A.thermal) B = B + P.sigma[beta] * normals3(thermal_bits(A.key, (uint32_t)i), T(0));
                    const V3<T> Ai = llg_A(mi, B, A.gp, A.alpha);
                    if constexpr (STAGE == PAIR_PREDICT) {
                        if (solver == SOLVER_HEUN) {
                            const V3<T> d = cross(mi, Ai);
                            store3(Abuf, N, i, d);
                            store3(out, N, i, normalize3(mi + A.dt * d));
                        } else if (solver == SOLVER_SIB) {
                            store3(out, N, i, T(0.5) * (mi + sib_stage(mi, Ai, A.dt)));
                        } else {
                            store3(Abuf, N, i, Ai);
                            store3(out, N, i, renorm_if_float(rotate(mi, T(-1) * Ai, A.dt)));
                        }
                    } else {
                        const V3<T> ni = load3(n, N, i);
                        if (solver == SOLVER_HEUN) {
                            const V3<T> d0 = load3(Abuf, N, i);
                            store3(out, N, i, normalize3(ni + (T(0.5) * A.dt) * (d0 + cross(mi, Ai))));
                        } else if (solver == SOLVER_SIB) {
                            store3(out, N, i, renorm_if_float(sib_stage(ni, Ai, A.dt)));
                        } else {
                            const V3<T> A0 = load3(Abuf, N, i);
                            store3(out, N, i, renorm_if_float(rotate(ni, T(-0.5) * (A0 + Ai), A.dt)));
                        }
                    }
                }
            }
        }
    }
    if constexpr (STAGE == PAIR_OBSERVE) {
        block_reduce(acc);
        if (tid == 0) {
#pragma unroll
            for (int k = 0; k < OBS_NVALS; ++k) partials[blockIdx.x * OBS_NVALS + k] = acc[k];
        }
    }
}

}  // namespace sp
