// kernels_dipole.hpp -- dipole-dipole gradient by direct summation over all
// pairs of the sample (the O(N^2) form of the dipolar term of the
// Hamiltonian, Sec. III.A):
//   g_dd_i = C_dd mu_i sum_{j != i} mu_j [n_j - 3 (n_j . r_ij) r_ij] / r_ij^3.
//
// Two forms, both with the S slice results summed in a fixed order by a
// second kernel:
//   k_dipole_partial  the interaction formed on the fly on the vector ALUs:
//                     workgroups own IPT*256 targets and one of S slices of
//                     the sources, staged 256 at a time in LDS (22.4 VALU
//                     instructions per pair, two-level summation);
//   k_dipole_mfma     the interaction tensor depends only on the translation
//                     between two sites, so it is tabulated once per
//                     Hamiltonian (formed in FP64) and the sum becomes, for
//                     each distance between rows, a matrix product on the
//                     matrix cores.
#pragma once

#include "device_common.hpp"

namespace sp {

// Lattice of an interaction table: A1, A2, A3, then the basis (Angstrom).
// Small enough to travel with a launch's arguments.
struct DipoleGeo {
    double v[9 + 3 * kMaxBasis];
};

template <typename T>
struct DipoleArgs {
    int N;
    int cells;           // sites per sublattice
    int slices;          // S
    int slice_len;       // sources per slice (multiple of 256)
    T mu[kMaxBasis];
};

// gate: when non-null and *gate == 0 the kernel does nothing (the surrogate's
// fallback launches the direct sum unconditionally and lets the device-side
// residual check decide).
template <typename T, int IPT>
__global__ void __launch_bounds__(256) k_dipole_partial(DipoleArgs<T> a, const T* __restrict__ pos,
                                                        const T* __restrict__ n, T* __restrict__ part,
                                                        const int* __restrict__ gate) {
    if (gate && *gate == 0) return;
    __shared__ T sp_[6][256];
    const int N = a.N;
    const int i0 = blockIdx.x * (256 * IPT) + threadIdx.x;
    T px[IPT], py[IPT], pz[IPT], gx[IPT], gy[IPT], gz[IPT];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        const int i = i0 + u * 256;
        const int ii = i < N ? i : N - 1;
        px[u] = pos[ii];
        py[u] = pos[N + ii];
        pz[u] = pos[2 * N + ii];
        gx[u] = gy[u] = gz[u] = T(0);
    }
    const int jbeg = blockIdx.y * a.slice_len;
    const int jend = min(N, jbeg + a.slice_len);
    for (int jt = jbeg; jt < jend; jt += 256) {
        __syncthreads();
        {
            const int j = jt + threadIdx.x;
            if (j < jend) {
                const T m = a.mu[j / a.cells];
                sp_[0][threadIdx.x] = pos[j];
                sp_[1][threadIdx.x] = pos[N + j];
                sp_[2][threadIdx.x] = pos[2 * N + j];
                sp_[3][threadIdx.x] = m * n[j];
                sp_[4][threadIdx.x] = m * n[N + j];
                sp_[5][threadIdx.x] = m * n[2 * N + j];
            } else {
                // zero moment: contributes exactly zero
                sp_[0][threadIdx.x] = T(0);
                sp_[1][threadIdx.x] = T(0);
                sp_[2][threadIdx.x] = T(0);
                sp_[3][threadIdx.x] = T(0);
                sp_[4][threadIdx.x] = T(0);
                sp_[5][threadIdx.x] = T(0);
            }
        }
        __syncthreads();
        T tx[IPT], ty[IPT], tz[IPT];
#pragma unroll
        for (int u = 0; u < IPT; ++u) tx[u] = ty[u] = tz[u] = T(0);
        for (int jj = 0; jj < 256; ++jj) {
            const T qx = sp_[0][jj], qy = sp_[1][jj], qz = sp_[2][jj];
            const T mx = sp_[3][jj], my = sp_[4][jj], mz = sp_[5][jj];
#pragma unroll
            for (int u = 0; u < IPT; ++u) {
                const T rx = qx - px[u], ry = qy - py[u], rz = qz - pz[u];
                const T d2 = rx * rx + ry * ry + rz * rz;
                T inv;
                if constexpr (sizeof(T) == 4) {
                    inv = d2 > T(0) ? __builtin_amdgcn_rsqf(d2) : T(0);
                } else {
                    inv = d2 > T(0) ? T(1) / sqrt(d2) : T(0);
                }
                const T inv2 = inv * inv;
                const T inv3 = inv2 * inv;
                const T s = T(3) * (mx * rx + my * ry + mz * rz) * inv2;
                tx[u] += (mx - s * rx) * inv3;
                ty[u] += (my - s * ry) * inv3;
                tz[u] += (mz - s * rz) * inv3;
            }
        }
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            gx[u] += tx[u];
            gy[u] += ty[u];
            gz[u] += tz[u];
        }
    }
    T* out = part + (size_t)blockIdx.y * 3 * N;
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        const int i = i0 + u * 256;
        if (i < N) {
            out[i] = gx[u];
            out[N + i] = gy[u];
            out[2 * N + i] = gz[u];
        }
    }
}

// ------------------------------------------------- matrix-core form
// With sites (a, b, plane p) the sum over the sources of one plane p2 in the
// rows b + db is, for a block of targets (a, b .. b + 15),
//   g^alpha[b][a] += sum_beta sum_a' m^beta[b + db][a'] K^{alpha beta}(a' - a; db, p, p2):
// a product of the spins of sixteen rows (M) with the Toeplitz matrix of one
// row distance (K x N), FP32 in FP32 accumulators (FP64 in FP64).  A
// wavefront owns 16 rows x 16 sites and three accumulators (alpha); nine
// 16x16x4 products per four sources.  A workgroup (WA wavefronts side by
// side along a) walks the units (source plane, chunk of KC source sites,
// row distance db) of its slice: per unit one new row of spins enters a ring
// of 32 rows in LDS and the six tensor components of the next distance are
// staged, both loaded while the current unit is multiplied.  Each unit is
// accumulated separately and then added (two-level summation).
// Bound: 9 x 32 cycles of matrix issue per 16 x 16 x 4 pairs against 22.4
// VALU instructions per pair of the other form; the padding to 16 sites and
// the Nb + 15 row distances of a 16-row block are its overhead.  Film of 128 x
// 128 x 4 sites: 1.95 ms per field with the vector form, 0.67 ms with this
// one (0.55 ms is the matrix rate of its padded products), error against 64 bits
// 3.2e-7 before and 2.5e-7 now.
template <typename T>
struct DipoleMfmaArgs {
    int N, Na, Nb, Nc, Nbas, P;
    int tiles_a, tiles_b, chunks;   // target tiles of 16 WA x 16 sites, source chunks
    int slices;
    int RL, pad;                    // table row length; entry of translation da = 0
    T mu[kMaxBasis];
};

template <typename T>
struct Mfma16;
template <>
struct Mfma16<float> {
    typedef float V __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mul(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int i) { return 4 * (lane >> 4) + i; }
};
template <>
struct Mfma16<double> {
    typedef double V __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mul(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int i) { return (lane >> 4) + 4 * i; }
};

constexpr int kDipChunk = 64;       // source sites of a row per unit

// Interaction table [offset][db + Nb - 1][component][RL]: component xx xy xz
// yy yz zz of (1 - 3 r^ r^) / r^3 with r the translation (da, db, c' - c)
// plus the basis difference; zero at r = 0 and beyond the sample.
template <typename T>
__global__ void __launch_bounds__(256) k_dipole_table(DipoleMfmaArgs<T> a, DipoleGeo G, T* __restrict__ K) {
    const double* geo = G.v;
    const int x = blockIdx.x * 256 + threadIdx.x;
    if (x >= a.RL) return;
    const int db = (int)blockIdx.y - (a.Nb - 1), off = blockIdx.z;
    const int nb2 = a.Nbas * a.Nbas;
    const int dc = off / nb2 - (a.Nc - 1), beta = (off % nb2) / a.Nbas, beta2 = off % a.Nbas;
    const int da = x - a.pad;
    T* o = K + ((size_t)off * (2 * a.Nb - 1) + blockIdx.y) * 6 * a.RL + x;
    double w[6] = {0, 0, 0, 0, 0, 0};
    if (da > -a.Na && da < a.Na) {
        double r[3];
        for (int k = 0; k < 3; ++k)
            r[k] = da * geo[k] + db * geo[3 + k] + dc * geo[6 + k] + geo[9 + 3 * beta2 + k] - geo[9 + 3 * beta + k];
        const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
        if (r2 > 1e-20) {
            const double inv = 1.0 / sqrt(r2), inv3 = inv * inv * inv;
            const double e[3] = {r[0] * inv, r[1] * inv, r[2] * inv};
            w[0] = (1.0 - 3.0 * e[0] * e[0]) * inv3;
            w[1] = -3.0 * e[0] * e[1] * inv3;
            w[2] = -3.0 * e[0] * e[2] * inv3;
            w[3] = (1.0 - 3.0 * e[1] * e[1]) * inv3;
            w[4] = -3.0 * e[1] * e[2] * inv3;
            w[5] = (1.0 - 3.0 * e[2] * e[2]) * inv3;
        }
    }
    for (int s = 0; s < 6; ++s) o[(size_t)s * a.RL] = (T)w[s];
}

// Grid: (tiles_a * tiles_b * P, slices), 64 WA threads.
template <typename T, int WA>
__global__ void __launch_bounds__(64 * WA) k_dipole_mfma(DipoleMfmaArgs<T> a, const T* __restrict__ K,
                                                         const T* __restrict__ n, T* __restrict__ part,
                                                         const int* __restrict__ gate) {
    if (gate && *gate == 0) return;
    using MM = Mfma16<T>;
    using V = typename MM::V;
    constexpr int KC = kDipChunk, AW = 16 * WA, NT = 64 * WA;
    constexpr int PITCH = KC + 4;                 // sixteen rows of four values meet different banks
    constexpr int KL = KC + AW;                   // tensor entries of a unit (the last is not used)
    __shared__ __align__(16) T ring[3][32][PITCH];
    __shared__ T kb[2][6][KL];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lk = lane >> 4;
    const int tile = blockIdx.x;
    const int ta = tile % a.tiles_a, tb = (tile / a.tiles_a) % a.tiles_b, p = tile / (a.tiles_a * a.tiles_b);
    const int a0 = ta * AW, b0 = tb * 16;
    const int c = p % a.Nc, beta = p / a.Nc;
    const int ndb = a.Nb + 15;                    // db = -(b0 + 15) .. Nb - 1 - b0
    const int units = a.P * a.chunks * ndb;
    const int u0 = (int)((long long)units * blockIdx.y / a.slices);
    const int u1 = (int)((long long)units * (blockIdx.y + 1) / a.slices);

    // unit u: source plane, first source site, row distance
    auto decode = [&](int u, int& p2, int& k0, int& db) {
        const int g = u / ndb;
        db = u - g * ndb - (b0 + 15);
        p2 = g / a.chunks;
        k0 = (g - p2 * a.chunks) * KC;
    };
    // moment component q of site (k0 + k) in row r of plane p2, zero outside
    auto moment = [&](int p2, int k0, int q, int r, int k) {
        if (r < 0 || r >= a.Nb || k0 + k >= a.Na) return T(0);
        return a.mu[p2 / a.Nc] * n[(size_t)q * a.N + ((size_t)p2 * a.Nb + r) * a.Na + k0 + k];
    };
    // first entry of the staged part of the table row of a unit; distances
    // beyond the sample (some rows of the block still have a partner) are
    // read from the nearest one: their products meet zero spins only
    auto row_of = [&](int p2, int k0, int db) {
        const int dc = p2 % a.Nc - c;
        const int off = ((dc + a.Nc - 1) * a.Nbas + beta) * a.Nbas + p2 / a.Nc;
        const int d = min(max(db, 1 - a.Nb), a.Nb - 1);
        return K + ((size_t)off * (2 * a.Nb - 1) + (d + a.Nb - 1)) * 6 * a.RL + a.pad + k0 - a0 - (AW - 1);
    };
    constexpr int KR = (6 * KL + NT - 1) / NT, MR = (3 * KC + NT - 1) / NT;
    V tot[3] = {V{0, 0, 0, 0}, V{0, 0, 0, 0}, V{0, 0, 0, 0}};
    bool fresh = true;      // the ring and tensor of this unit are not staged
    int cur = 0;
    for (int u = u0; u < u1; ++u) {
        int p2, k0, db;
        decode(u, p2, k0, db);
        if (fresh) {
            __syncthreads();
            for (int t = tid; t < 3 * 16 * KC; t += NT) {
                const int k = t % KC, j = (t / KC) & 15, q = t / (16 * KC);
                const int r = b0 + db + j;
                ring[q][r & 31][k] = moment(p2, k0, q, r, k);
            }
            const T* src = row_of(p2, k0, db);
            for (int t = tid; t < 6 * KL; t += NT) kb[cur][t / KL][t % KL] = src[(size_t)(t / KL) * a.RL + t % KL];
            __syncthreads();
        }
        // the next unit's new row and tensor, on their way during the product
        const bool more = u + 1 < u1 && (u + 1) % ndb != 0;
        T pk[KR], pm[MR];
        if (more) {
            const T* src = row_of(p2, k0, db + 1);
#pragma unroll
            for (int i = 0; i < KR; ++i) {
                const int t = tid + i * NT;
                if (t < 6 * KL) pk[i] = src[(size_t)(t / KL) * a.RL + t % KL];
            }
#pragma unroll
            for (int i = 0; i < MR; ++i) {
                const int t = tid + i * NT;
                if (t < 3 * KC) pm[i] = moment(p2, k0, t / KC, b0 + db + 16, t % KC);
            }
        }
        const int slot = (b0 + db + l16) & 31;
        const T(*kk)[KL] = kb[cur];
        const int j0 = 4 * lk - (16 * wave + l16) + AW - 1;
        const int steps = (min(KC, a.Na - k0) + 15) / 16;
        V acc[3] = {V{0, 0, 0, 0}, V{0, 0, 0, 0}, V{0, 0, 0, 0}};
        for (int s = 0; s < steps; ++s) {
            // sources 16 s + 4 lk .. + 3 of this lane's quarter
            T m[3][4];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const T* r = &ring[q][slot][16 * s + 4 * lk];
#pragma unroll
                for (int i = 0; i < 4; ++i) m[q][i] = r[i];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = j0 + 16 * s + i;
                const T xx = kk[0][j], xy = kk[1][j], xz = kk[2][j], yy = kk[3][j], yz = kk[4][j], zz = kk[5][j];
                acc[0] = MM::mul(m[0][i], xx, acc[0]);
                acc[1] = MM::mul(m[0][i], xy, acc[1]);
                acc[2] = MM::mul(m[0][i], xz, acc[2]);
                acc[0] = MM::mul(m[1][i], xy, acc[0]);
                acc[1] = MM::mul(m[1][i], yy, acc[1]);
                acc[2] = MM::mul(m[1][i], yz, acc[2]);
                acc[0] = MM::mul(m[2][i], xz, acc[0]);
                acc[1] = MM::mul(m[2][i], yz, acc[1]);
                acc[2] = MM::mul(m[2][i], zz, acc[2]);
            }
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) tot[q] += acc[q];
        fresh = !more;
        if (more) {
            cur ^= 1;
#pragma unroll
            for (int i = 0; i < KR; ++i) {
                const int t = tid + i * NT;
                if (t < 6 * KL) kb[cur][t / KL][t % KL] = pk[i];
            }
#pragma unroll
            for (int i = 0; i < MR; ++i) {
                const int t = tid + i * NT;
                if (t < 3 * KC) ring[t / KC][(b0 + db + 16) & 31][t % KC] = pm[i];
            }
            __syncthreads();
        }
    }
    T* out = part + (size_t)blockIdx.y * 3 * a.N;
    const int ai = a0 + 16 * wave + l16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int bi = b0 + MM::row(lane, i);
        if (ai < a.Na && bi < a.Nb) {
            const size_t o = ((size_t)p * a.Nb + bi) * a.Na + ai;
#pragma unroll
            for (int q = 0; q < 3; ++q) out[(size_t)q * a.N + o] = tot[q][i];
        }
    }
}

// Sum the S slices in order and scale by C_dd mu_i.
template <typename T>
__global__ void __launch_bounds__(256) k_dipole_finish(DipoleArgs<T> a, T Cdd, const T* __restrict__ part,
                                                       T* __restrict__ gdd, const int* __restrict__ gate) {
    if (gate && *gate == 0) return;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int N = a.N;
    if (t >= 3 * N) return;
    const int i = t % N;
    // eight slices in flight, added in order
    T s = T(0);
    for (int k0 = 0; k0 < a.slices; k0 += 8) {
        T v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = part[(size_t)min(k0 + k, a.slices - 1) * 3 * N + t];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k0 + k < a.slices) s += v[k];
    }
    gdd[t] = Cdd * a.mu[i / a.cells] * s;
}

}  // namespace sp
