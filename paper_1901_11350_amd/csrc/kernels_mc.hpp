// kernels_mc.hpp -- Metropolis Monte Carlo with cone trial moves (Sec. III.B).
// The paper's sweep picks every spin once, one after another, in random
// order.  Here a sweep is a multi-colour pass: the host colours the sites
// periodically -- colour(i) = table[a mod ma][b mod mb][c mod mc][beta] --
// so that no bond joins two sites of one colour (two colours, the
// checkerboard, for the simple-cubic nearest-neighbour lattice; three or
// more for triangular, second-neighbour or basis lattices), and one launch
// updates a whole colour in parallel; every site is still tried once per
// sweep and each trial sees the current state of every spin it interacts
// with, so the chain samples the same Boltzmann distribution (checked
// statistically against the sequential random-order sweep).
//
// Trial at site i of sweep s: Philox block of counter (i, s_lo, s_hi,
// replica), u_k = (x_k + 1/2) 2^-32; phi = 2 pi u0, cos(theta) = 1 - u1 (1 -
// cos(cone)); new spin cos(theta) n + sin(theta) (cos(phi) e1 + sin(phi) e2),
// e1 = unit(n x r) with r = z if |n_z| < 0.9 else x, e2 = n x e1; accepted
// if u2 < exp(-dE / k_B T).  dE needs only the terms containing site i:
// Zeeman and the pair terms are linear in n_i (dn . coefficient), the
// anisotropy and the on-site Gaussians are evaluated at both spins.
// Adaptive cone: after every sweep the cone is multiplied by
// 1 + a - a* (a the sweep's acceptance ratio, a* the target), at most 180
// degrees, on the device.
#pragma once

#include "kernels_pairs.hpp"

namespace sp {

struct McClass;

template <typename T>
struct McArgs {
    T kT;            // k_B T (meV)
    T cos_cone;
    ThermalKey key;  // seed, sweep number (step words), replica
    const double* cone_dev;   // adaptive cone (degrees) on the device, or null: cos_cone
    const McClass* cls;       // the classes of the colour
    int n_cls;
    int start[8];             // first workgroups of up to eight classes
    int cm[3];                // periods of the colouring
    int near, dmi;            // every offset shorter than its periodic axis; some bond has a DMI vector
};

// The sites of one class (a mod cm[0], b mod cm[1], c mod cm[2], beta): n[k]
// of them along axis k from first[k] on, with bonds q0 to q1 - 1; its
// workgroups start at block.
struct McClass {
    int first[3], beta, n[3], block, q0, q1;
};

template <typename T>
__device__ __forceinline__ void mc_uniforms(const U4& x, T u[3]) {
    if constexpr (sizeof(T) == 4) {
        u[0] = fmaf((float)x.x, 0x1p-32f, 0x1p-33f);
        u[1] = fmaf((float)x.y, 0x1p-32f, 0x1p-33f);
        u[2] = fmaf((float)x.z, 0x1p-32f, 0x1p-33f);
    } else {
        u[0] = ((double)x.x + 0.5) * 0x1p-32;
        u[1] = ((double)x.y + 0.5) * 0x1p-32;
        u[2] = ((double)x.z + 0.5) * 0x1p-32;
    }
}

template <typename T>
__device__ __forceinline__ V3<T> mc_trial(V3<T> n, const T u[3], T cos_cone) {
    const V3<T> r = fabs(n.z) < T(0.9) ? V3<T>{T(0), T(0), T(1)} : V3<T>{T(1), T(0), T(0)};
    const V3<T> e1 = normalize3(cross(n, r));
    const V3<T> e2 = cross(n, e1);
    T sp, cp;
    if constexpr (sizeof(T) == 4) {
        sp = __builtin_amdgcn_sinf(u[0]);   // argument in revolutions
        cp = __builtin_amdgcn_cosf(u[0]);
    } else {
        sincospi(T(2) * u[0], &sp, &cp);
    }
    const T ct = T(1) - u[1] * (T(1) - cos_cone);
    const T st = sqrt(fmax(T(0), T(1) - ct * ct));
    return V3<T>{ct * n.x + st * (cp * e1.x + sp * e2.x), ct * n.y + st * (cp * e1.y + sp * e2.y),
                 ct * n.z + st * (cp * e1.z + sp * e2.z)};
}

// Exchange and DMI sums of the site (a, b, c), its bonds q0 to q1 - 1 uniform
// over the workgroup, in the order of site_terms.  G bonds at a time: their
// records are read together (scalar), then their neighbours, then their
// couplings under the neighbours' latency.  NEAR: no offset reaches past one
// lattice length of a periodic axis, so a wrap is two selects; with the
// division of the general case in the loop its branches kept every record's
// load behind the one before (6.9 -> 6.0 us per colour of 30^3 sites).  DMI: the vectors are read.
template <typename T, bool NEAR, bool DMI, int G>
__device__ __forceinline__ void mc_pair_sums(const Lattice& L, const BondCoef<double>& C, const T* __restrict__ n, int a,
                                             int b, int c, int q0, int q1, int i, V3<double>& gj, V3<double>& gd) {
    auto coord = [](int t, int len, int per, bool& ok) {
        if constexpr (!NEAR) return frame_coord(t, len, per, ok);
        const int w = t < 0 ? t + len : (t >= len ? t - len : t);
        ok = ok && (per != 0 || w == t);
        return w;
    };
    for (int q = q0; q < q1; q += G) {
        int4 bd[G];
        V3<T> v[G];
#pragma unroll
        for (int u = 0; u < G; ++u) bd[u] = L.bond[min(q + u, q1 - 1)];
#pragma unroll
        for (int u = 0; u < G; ++u) asm volatile("" ::"s"(bd[u].x), "s"(bd[u].y), "s"(bd[u].z), "s"(bd[u].w));
#pragma unroll
        for (int u = 0; u < G; ++u) {
            bool ok = q + u < q1;
            const int ta = coord(a + bd[u].y, L.n[0], L.per[0], ok);
            const int tb = coord(b + bd[u].z, L.n[1], L.per[1], ok);
            const int tc = coord(c + bd[u].w, L.n[2], L.per[2], ok);
            v[u] = load3(n, L.N, ok ? ta + L.n[0] * (tb + L.n[1] * (tc + L.n[2] * bd[u].x)) : i);
            if (!ok) v[u] = V3<T>{T(0), T(0), T(0)};
        }
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int k = min(q + u, q1 - 1);
            const double J = C.J[k];
            const V3<double> nj{(double)v[u].x, (double)v[u].y, (double)v[u].z};
            gj = gj - J * nj;
            if constexpr (DMI) gd = gd - cross(nj, V3<double>{C.D[3 * k], C.D[3 * k + 1], C.D[3 * k + 2]});
        }
    }
}

template <typename T>
__device__ __forceinline__ void mc_pair_terms(const Lattice& L, const BondCoef<double>& C, const T* __restrict__ n, int a,
                                              int b, int c, int q0, int q1, int i, bool near, bool dmi, V3<double>& gj,
                                              V3<double>& gd) {
    gj = gd = V3<double>{0.0, 0.0, 0.0};
    // six at a time, or four where that leaves fewer places empty: a launch of
    // few sites is one wavefront's chain, and an empty place costs it as much
    // as a bond (64 sites of four bonds, 100 sweeps: 1351 us by sixes, 1264 by
    // fours; 1024^2 sites, 20 sweeps: 885 and 819)
    const int count = q1 - q0;
    const bool four = (count + 3) / 4 * 4 < (count + 5) / 6 * 6;
    if (!near) mc_pair_sums<T, false, true, 6>(L, C, n, a, b, c, q0, q1, i, gj, gd);
    else if (dmi && four) mc_pair_sums<T, true, true, 4>(L, C, n, a, b, c, q0, q1, i, gj, gd);
    else if (dmi) mc_pair_sums<T, true, true, 6>(L, C, n, a, b, c, q0, q1, i, gj, gd);
    else if (four) mc_pair_sums<T, true, false, 4>(L, C, n, a, b, c, q0, q1, i, gj, gd);
    else mc_pair_sums<T, true, false, 6>(L, C, n, a, b, c, q0, q1, i, gj, gd);
}

// One colour of one sweep: a workgroup takes sites of one class of the
// colour, every lane a site.  (A launch over all sites that tested each one's
// colour left half or more of the lanes idle and read bond after bond from
// per-lane lists: 8.2 us per colour of 30^3 sites.)  acc_part[block]
// accumulates the accepted trials of this workgroup over the launches of a
// run.  The accept/reject decision is taken in FP64 for every engine
// precision (the precision of the FP64 reference): trial spin, energy
// difference and Metropolis test from the stored spins (type T) with FP64
// couplings; an accepted trial is stored rounded to T.
template <typename T>
__global__ void __launch_bounds__(256) k_mc_colour(Lattice L, BondCoef<double> C, Phys<double> P,
                                                   McArgs<double> M, T* __restrict__ n,
                                                   unsigned int* __restrict__ acc_part) {
    unsigned int acc0 = 0;
    if (threadIdx.x == 0) acc0 = acc_part[blockIdx.x];
    // the class of this workgroup: the last that starts at or before it (a
    // search in memory is a load after a load, so few classes bring their
    // starts with the arguments)
    int lo = 0;
    if (M.n_cls <= 8) {
#pragma unroll
        for (int k = 1; k < 8; ++k)
            if (k < M.n_cls && M.start[k] <= (int)blockIdx.x) lo = k;
    } else {
        int hi = M.n_cls - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (M.cls[mid].block <= (int)blockIdx.x) lo = mid;
            else hi = mid - 1;
        }
    }
    const McClass K = M.cls[lo];
    const int t = ((int)blockIdx.x - K.block) * (int)blockDim.x + (int)threadIdx.x;
    bool accepted = false;
    if (t < K.n[0] * K.n[1] * K.n[2]) {
        const int r = t / K.n[0], kc = r / K.n[1];
        const int a = K.first[0] + M.cm[0] * (t - r * K.n[0]);
        const int b = K.first[1] + M.cm[1] * (r - kc * K.n[1]);
        const int c = K.first[2] + M.cm[2] * kc;
        const int beta = K.beta;
        const int i = a + L.n[0] * (b + L.n[1] * (c + L.n[2] * beta));
        const V3<T> st = load3(n, L.N, i);
        V3<double> gj, gd;
        mc_pair_terms(L, C, n, a, b, c, K.q0, K.q1, i, M.near != 0, M.dmi != 0, gj, gd);
        asm volatile("" ::"v"(acc0));   // its load has come in with the neighbours'
        const V3<double> ni{(double)st.x, (double)st.y, (double)st.z};
        double u[3];
        mc_uniforms<double>(thermal_bits(M.key, (uint32_t)i), u);
        const double cos_cone = M.cone_dev ? cos(*M.cone_dev * (3.141592653589793 / 180.0)) : M.cos_cone;
        const V3<double> nn = mc_trial(ni, u, cos_cone);
        const V3<double> gz{P.gZ[beta][0], P.gZ[beta][1], P.gZ[beta][2]};
        const V3<double> lin = gz + gj + gd;
        const V3<double> ax{P.Kax[beta][0], P.Kax[beta][1], P.Kax[beta][2]};
        const double k0 = dot(ax, ni), k1 = dot(ax, nn);
        const double dE = dot(nn - ni, lin) - 0.5 * P.K2[beta] * (k1 * k1 - k0 * k0) +
                          (gauss_energy(P, nn) - gauss_energy(P, ni));
        if (u[2] < exp(-dE / M.kT)) {
            store3(n, L.N, i, V3<T>{(T)nn.x, (T)nn.y, (T)nn.z});
            accepted = true;
        }
    }
    const unsigned long long mask = __ballot(accepted);
    __shared__ unsigned int cnt[4];
    if ((threadIdx.x & 63) == 0) cnt[threadIdx.x >> 6] = (unsigned int)__popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned int s = 0;
        for (int w = 0; w < (int)blockDim.x >> 6; ++w) s += cnt[w];
        acc_part[blockIdx.x] = acc0 + s;
    }
}

// Feedback of the adaptive cone after one sweep: the sweep's accepted trials
// are the growth of the run's per-workgroup counts (summed in a fixed
// order) since the previous sweep; state[0] is the cone in degrees,
// state[1] the count at the previous sweep.
__global__ void __launch_bounds__(256) k_mc_adapt(const unsigned int* __restrict__ acc_part, int blocks,
                                                  long long n_sites, double target, double* __restrict__ state) {
    __shared__ unsigned long long red[256];
    unsigned long long t = 0;
    for (int b = threadIdx.x; b < blocks; b += 256) t += acc_part[b];
    red[threadIdx.x] = t;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double total = (double)red[0];
        const double a = n_sites > 0 ? (total - state[1]) / (double)n_sites : 0.0;
        const double c = state[0] * (1.0 + a - target);
        state[0] = c > 180.0 ? 180.0 : c;
        state[1] = total;
    }
}

}  // namespace sp
