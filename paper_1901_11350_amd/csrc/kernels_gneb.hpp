// kernels_gneb.hpp -- geodesic nudged elastic band on the GPU (Sec. III.D;
// Appendix F for tangents, distances and projections; Appendix D for the
// velocity-projection minimiser).
//
// The chain holds M images of N spins, image-major, each image SoA.  Images 0
// and M-1 are fixed.  Between iterations the minimiser's state is the chain,
// the force F of the last evaluation and the partials of v.F and F.F: the
// projected velocity is v = (v.F/F.F) F if v.F > 0 else 0, a multiple of F,
// so no velocity array exists.  Per velocity-projection iteration:
//   k_gneb_grad_tile  s = v.F/F.F from the partials, then on tiles of the
//                     image: x <- normalise(x + dt s F + dt^2/(2m) F) (into
//                     the other chain buffer), g = dH/dn, energy partials
//                     (k_gneb_move in place and k_gneb_grad on lattices
//                     without a compile-time 2D stencil)
//   k_gneb_tangent    E of the image and its neighbours from the partials;
//                     improved tangent, per-spin projection; partials of
//                     |tau|^2, g.tau, and squared geodesic angles to image v+1
//   k_gneb_force      |tau|^2, g.tau, l^2 from the partials; the tangent
//                     again (two multiply-adds a component, against storing
//                     and loading it);
//                     F = -g + (g.t)t, per-spin projected, + k (l_v - l_{v-1}) t
//                     (climbing images: -g + 2 (g.t)t, falling: -g, no spring)
//                     with t = tau/|tau|; partials of v.F and F.F with
//                     v <- s F_prev + dt/(2m)(F_prev + F)
// The last two walk several images per workgroup, so a chain's arrays are
// read about once each; k_gneb_sum adds the partials of large chains, whose
// every workgroup would otherwise spend its time on them.
// Every reduction is a fixed-order FP64 tree: a row of partials is summed by
// the same strided loop and tree in every workgroup that needs it
// (bit-reproducible, identical everywhere).
// What bounds it: about 7 passes over arrays that stay in the last-level
// cache, and the latency of three dependent launches.  On 32 images of
// 128^2 spins (FP32) six launches with stored velocity, previous force and
// tangent took 45 us per iteration, these three 30.
#pragma once

#include "kernels_field.hpp"
#include "kernels_reduce.hpp"
#include "kernels_stencil.hpp"

namespace sp {

template <int NV>
__device__ __forceinline__ void block_sums(double* acc) {
    __shared__ double red[4][NV];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const double v = wave_sum(acc[k]);
        if (lane == 0) red[wave][k] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[k] = red[0][k] + red[1][k] + red[2][k] + red[3][k];
    }
}

// Sum of row `row` of NV-value partials (nblk per row) by one wavefront,
// fixed order; every lane receives the result.
template <int NV>
__device__ __forceinline__ void wave_row_sum(const double* __restrict__ part, int nblk, int row, double* out) {
#pragma unroll
    for (int k = 0; k < NV; ++k) out[k] = 0.0;
    for (int b = threadIdx.x & 63; b < nblk; b += 64) {
#pragma unroll
        for (int k = 0; k < NV; ++k) out[k] += part[((size_t)row * nblk + b) * NV + k];
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) out[k] = wave_sum(out[k]);
}

// Velocity scale s = v.F / F.F (0 unless both are positive) from `count`
// partials; every thread receives it.
__device__ __forceinline__ double gneb_scale(const double* __restrict__ part, int count) {
    double acc[2] = {0.0, 0.0};
    for (int b0 = threadIdx.x; b0 < count; b0 += 4 * 256) {
        double v[4][2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int b = b0 + k * 256;
            v[k][0] = b < count ? part[2 * b] : 0.0;
            v[k][1] = b < count ? part[2 * b + 1] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            acc[0] += v[k][0];
            acc[1] += v[k][1];
        }
    }
    block_sums<2>(acc);
    __shared__ double bc;
    if (threadIdx.x == 0) bc = acc[0] > 0.0 && acc[1] > 0.0 ? acc[0] / acc[1] : 0.0;
    __syncthreads();
    return bc;
}

// Weights of the improved tangent towards the next and the previous image.
__device__ __forceinline__ void gneb_weights(double Em, double E0, double Ep, double& wp, double& wm) {
    if (Ep > E0 && E0 > Em) {
        wp = 1.0; wm = 0.0;
    } else if (Ep < E0 && E0 < Em) {
        wp = 0.0; wm = 1.0;
    } else {
        const double d1 = fabs(Ep - E0), d2 = fabs(Em - E0);
        const double dmax = d1 > d2 ? d1 : d2, dmin = d1 > d2 ? d2 : d1;
        if (Ep > Em) { wp = dmax; wm = dmin; } else { wp = dmin; wm = dmax; }
    }
}

// Tangent of one spin, unnormalised, projected onto its tangent plane.
template <typename T>
__device__ __forceinline__ V3<T> gneb_tau(V3<T> nm, V3<T> n0, V3<T> np, double wp, double wm) {
    const V3<T> t = T(wp) * (np - n0) + T(wm) * (n0 - nm);
    return t - dot(t, n0) * n0;
}

// Maximum over the block (thread 0 receives it).
__device__ __forceinline__ double block_max(double v) {
    __shared__ double red[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_max(v);
    if (lane == 0) red[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) v = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    return v;
}

struct GnebDims {
    int M;         // images
    int N;         // spins per image
    int nblk;      // blocks per image in the per-site kernels
    int nblk_e;    // energy partials per image (blocks of the gradient kernel)
};

// Position step of one spin: x + dt v + dt^2/(2m) F with v = scale F,
// renormalised.
template <typename T>
__device__ __forceinline__ V3<T> gneb_moved(V3<T> x, V3<T> f, T scale, T dt, T half_dt2_m) {
    const T n0 = x.x + dt * (scale * f.x) + half_dt2_m * f.x;
    const T n1 = x.y + dt * (scale * f.y) + half_dt2_m * f.y;
    const T n2 = x.z + dt * (scale * f.z) + half_dt2_m * f.z;
    const T r = T(1) / sqrt(n0 * n0 + n1 * n1 + n2 * n2);
    return V3<T>{n0 * r, n1 * r, n2 * r};
}

// The position step alone, in place (interior images).
template <typename T>
__global__ void __launch_bounds__(256) k_gneb_move(GnebDims d, T dt, T half_dt2_m, const double* __restrict__ part,
                                                   int parts, double* __restrict__ scale_out,
                                                   const T* __restrict__ F, T* __restrict__ x,
                                                   const int* __restrict__ stop) {
    if (stop && *stop) return;   // the chain has converged: the rest of the run is skipped
    const double sc = gneb_scale(part, parts);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *scale_out = sc;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= d.N) return;
    const size_t off = (size_t)(blockIdx.y + 1) * 3 * d.N;
    store3(x + off, d.N, i, gneb_moved(load3(x + off, d.N, i), load3(F + off, d.N, i), (T)sc, dt, half_dt2_m));
}

// Gradient of every image and per-block energy partials (Zeeman linear,
// the other local terms quadratic: e_i = n.(g_Z + (g_K + g_J + g_D)/2)).
template <typename T>
__global__ void __launch_bounds__(256) k_gneb_grad(GnebDims d, Lattice L, BondCoef<double> C, Phys<double> P,
                                                   const T* __restrict__ x, T* __restrict__ g,
                                                   double* __restrict__ part, int im0,
                                                   const int* __restrict__ stop) {
    if (stop && *stop) return;   // the chain has converged: the rest of the run is skipped
    // field and energy in FP64 from the stored spins (type T): the image
    // energies decide the tangent's branch, so they are formed in the
    // reference's precision for both engine precisions; g is stored as T
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int im = im0 + blockIdx.y;
    const T* xi = x + (size_t)im * 3 * d.N;
    double acc[1] = {0.0};
    if (i < d.N) {
        const V3<double> ni{(double)xi[i], (double)xi[d.N + i], (double)xi[2 * d.N + i]};
        const FieldTerms<double> f = site_terms<double, T>(L, C, P, xi, i, ni);
        const V3<double> gt = total(f);
        store3(g + (size_t)im * 3 * d.N, d.N, i, V3<T>{(T)gt.x, (T)gt.y, (T)gt.z});
        acc[0] = ni.x * f.z.x + ni.y * f.z.y + ni.z * f.z.z +
                 0.5 * (ni.x * (f.k.x + f.j.x + f.d.x) + ni.y * (f.k.y + f.j.y + f.d.y) +
                        ni.z * (f.k.z + f.j.z + f.d.z)) +
                 gauss_energy(P, ni);
    }
    block_sums<1>(acc);
    if (threadIdx.x == 0) part[(size_t)im * d.nblk_e + blockIdx.x] = acc[0];
}

// The same on TS x TS tiles of one-atom 2D images with a compile-time
// stencil (ragged tiles allowed), after the position step when MOVE: the
// tile and its R halo are stepped on the way into LDS (FP64 cells) and the
// tile's own spins stored to the other chain buffer.  Squares have the
// smallest halo.  Bound by instructions, so large chains take 32 x 32 tiles,
// four sites per thread: the halo is 1.13 times the tile (16 x 16: 1.27) and
// the velocity scale and the energy sum are formed a quarter as often; 16 x
// 16 where those would leave CUs without work.  The terms are those of
// shape_terms, in FP64 from the spins as stored.
template <typename T, int S, int NDMI, bool MOVE, int TS>
__global__ void __launch_bounds__(256)
    k_gneb_grad_tile(GnebDims d, ShapeCoef<double> C, Site2D<double> Q, int tiles_x, T dt, T half_dt2_m,
                     const double* __restrict__ fpart, int parts, double* __restrict__ scale_out,
                     const T* __restrict__ F, const T* __restrict__ x, T* __restrict__ xn, T* __restrict__ g,
                     double* __restrict__ part, int im0, const int* __restrict__ stop) {
    if (stop && *stop) return;   // the chain has converged: the rest of the run is skipped
    constexpr int TX = TS, TY = TS, NT = 256, SITES = TS * TS / NT;
    constexpr int R = ShapeTab<S>::R, W = TX + 2 * R, H = TY + 2 * R, P = W * H, KST = (P + NT - 1) / NT;
    __shared__ V4<double> sN[P];
    const int im = im0 + blockIdx.y, tile = blockIdx.x;
    const int tyi = tile / tiles_x;
    const int x0 = (tile - tyi * tiles_x) * TX, y0 = tyi * TY;
    const int N = d.N, tid = threadIdx.x;
    const size_t off = (size_t)im * 3 * N;
    V3<T> st[KST], sf[KST];
    int site[KST];               // the cell's site, or -1 outside an open lattice
    bool own[KST];
#pragma unroll
    for (int k = 0; k < KST; ++k) {
        const int idx = tid + k * NT;
        site[k] = -1;
        own[k] = false;
        st[k] = sf[k] = V3<T>{T(0), T(0), T(0)};
        if (idx < P) {
            const int ly = idx / W, lx = idx - ly * W;
            bool in = true;
            const int ux = x0 - R + lx, uy = y0 - R + ly;
            const int gx = wrap_once(ux, Q.na, Q.per_a, in);
            const int gy = wrap_once(uy, Q.nb, Q.per_b, in);
            if (in) {
                site[k] = gx + gy * Q.na;
                own[k] = lx >= R && lx < R + TX && ly >= R && ly < R + TY && ux < Q.na && uy < Q.nb;
                st[k] = load3(x + off, N, site[k]);
                if (MOVE) sf[k] = load3(F + off, N, site[k]);
            }
        }
    }
    T scale = T(0);
    if constexpr (MOVE) {
        const double sc = gneb_scale(fpart, parts);
        if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *scale_out = sc;
        scale = (T)sc;
    }
#pragma unroll
    for (int k = 0; k < KST; ++k) {
        const int idx = tid + k * NT;
        if (idx < P) {
            V4<double> cell{0.0, 0.0, 0.0, 0.0};
            if (site[k] >= 0) {
                V3<T> s = st[k];
                if constexpr (MOVE) {
                    s = gneb_moved(s, sf[k], scale, dt, half_dt2_m);
                    if (own[k]) store3(xn + off, N, site[k], s);
                }
                cell = V4<double>{(double)s.x, (double)s.y, (double)s.z, 0.0};
            }
            sN[idx] = cell;
        }
    }
    __syncthreads();
    double acc[1] = {0.0};
#pragma unroll
    for (int k = 0; k < SITES; ++k) {
        const int u = tid + k * NT;
        const int ty = u / TX, tx = u - ty * TX;
        const int gx = x0 + tx, gy = y0 + ty;
        if (gx < Q.na && gy < Q.nb) {
            const int c = (ty + R) * W + (tx + R);
            const V3<double> ni = lds_cell_xyz(sN, c);
            const FieldTerms<double> f = shape_terms<double, S, NDMI, W>(C, Q, sN, c, ni);
            const V3<double> gt = f.z + f.k + f.j + f.d;
            store3(g + off, N, gx + gy * Q.na, V3<T>{(T)gt.x, (T)gt.y, (T)gt.z});
            acc[0] += ni.x * f.z.x + ni.y * f.z.y + ni.z * f.z.z +
                      0.5 * (ni.x * (f.k.x + f.j.x + f.d.x) + ni.y * (f.k.y + f.j.y + f.d.y) +
                             ni.z * (f.k.z + f.j.z + f.d.z));
        }
    }
    block_sums<1>(acc);
    if (tid == 0) part[(size_t)im * d.nblk_e + tile] = acc[0];
}

// Sum NV-value partials of each of `rows` rows (blocks per row = nblk) in a
// fixed order: out[row*NV + k].
template <int NV>
__global__ void __launch_bounds__(256) k_gneb_sum(const double* __restrict__ part, int nblk, double* __restrict__ out,
    const int* __restrict__ stop) {
    if (stop && *stop) return;   // the chain has converged: the rest of the run is skipped
    const int row = blockIdx.x;
    double acc[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) acc[k] = 0.0;
    for (int b = threadIdx.x; b < nblk; b += 256) {
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[k] += part[((size_t)row * nblk + b) * NV + k];
    }
    block_sums<NV>(acc);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) out[row * NV + k] = acc[k];
    }
}

// Partials of |tau|^2, g.tau (interior images) and of the squared
// great-circle angle to the next image, for the IPW images from
// blockIdx.y * IPW (images 0 .. M - 2); E of every image.  All spins and
// gradients of the thread's site are loaded together.
template <typename T, int IPW>
__global__ void __launch_bounds__(256) k_gneb_tangent(GnebDims d, const T* __restrict__ x, const T* __restrict__ g,
                                                      const double* __restrict__ epart, double* __restrict__ E,
                                                      double* __restrict__ part, const int* __restrict__ stop) {
    if (stop && *stop) return;   // the chain has converged: the rest of the run is skipped
    __shared__ double sE[IPW + 2];
    __shared__ double red[IPW][3][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = blockIdx.x * 256 + tid;
    const int im0 = blockIdx.y * IPW, im1 = min(im0 + IPW, d.M - 1);
    const size_t L3 = (size_t)3 * d.N;
    const int ic = min(i, d.N - 1);
    V3<T> xs[IPW + 2], gs[IPW];      // images im0 - 1 .. im0 + IPW
#pragma unroll
    for (int k = 0; k < IPW + 2; ++k) xs[k] = load3(x + min(max(im0 - 1 + k, 0), d.M - 1) * L3, d.N, ic);
#pragma unroll
    for (int k = 0; k < IPW; ++k) gs[k] = load3(g + min(im0 + k, d.M - 1) * L3, d.N, ic);
    // energies of images im0 - 1 .. im1
    for (int r = max(im0 - 1, 0) + wave; r <= im1; r += 4) {
        double e;
        wave_row_sum<1>(epart, d.nblk_e, r, &e);
        if (lane == 0) {
            sE[r - im0 + 1] = e;
            if (blockIdx.x == 0 && (r >= im0 && (r < im1 || r == d.M - 1))) E[r] = e;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < IPW; ++k) {
        const int im = im0 + k;
        if (im >= im1) break;
        double acc[3] = {0.0, 0.0, 0.0};
        if (i < d.N) {
            const V3<T> c = cross(xs[k + 1], xs[k + 2]);
            // angle in working precision (its inputs are), squared sum in FP64
            const double ang = (double)atan2(sqrt(dot(c, c)), dot(xs[k + 1], xs[k + 2]));
            acc[2] = ang * ang;
            if (im > 0) {
                double wp, wm;
                gneb_weights(sE[k], sE[k + 1], sE[k + 2], wp, wm);
                const V3<T> t = gneb_tau(xs[k], xs[k + 1], xs[k + 2], wp, wm);
                acc[0] = (double)dot(t, t);
                acc[1] = (double)dot(gs[k], t);
            }
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const double v = wave_sum(acc[q]);
            if (lane == 0) red[k][q][wave] = v;
        }
    }
    __syncthreads();
    const int nv = (im1 - im0) * 3;
    if (tid < nv) {
        const double* r = red[tid / 3][tid % 3];
        part[((size_t)(im0 + tid / 3) * d.nblk + blockIdx.x) * 3 + tid % 3] = r[0] + r[1] + r[2] + r[3];
    }
}

// Forces of the IPW interior images from 1 + blockIdx.y * IPW (over the
// previous forces), partials of v.F and F.F with the velocity that follows
// (update_v; v.F = 0 otherwise).  s3[v] = (|tau|^2, g.tau, l^2).
// Image types: 0 normal, 1 climbing (no spring, F = -g + 2 (g.t) t),
// 2 falling (no spring, F = -g); all per-spin projected.
template <typename T, int IPW>
__global__ void __launch_bounds__(256) k_gneb_force(GnebDims d, T k_spring, T dt_2m, int update_v,
                                                    const double* __restrict__ scale, const T* __restrict__ x,
                                                    const T* __restrict__ g, const double* __restrict__ E,
                                                    const double* __restrict__ tpart, double* __restrict__ s3,
                                                    const int* __restrict__ types, T* __restrict__ F,
                                                    double* __restrict__ part, double* __restrict__ fmax_part,
                                                    const int* __restrict__ stop) {
    if (stop && *stop) return;   // the chain has converged: the rest of the run is skipped
    // per image: 1 / |tau|, g.t (times 2 or 0 by type), spring force, weights
    __shared__ double s[IPW + 1][3];
    __shared__ double inv_s[IPW], wp_s[IPW], wm_s[IPW];
    __shared__ T gt_s[IPW], fs_s[IPW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = blockIdx.x * 256 + tid;
    const int im0 = 1 + blockIdx.y * IPW, im1 = min(im0 + IPW, d.M - 1);
    const size_t L3 = (size_t)3 * d.N;
    const int ic = min(i, d.N - 1);
    V3<T> xs[IPW + 2], gs[IPW], fp[IPW];
#pragma unroll
    for (int k = 0; k < IPW + 2; ++k) xs[k] = load3(x + min(im0 - 1 + k, d.M - 1) * L3, d.N, ic);
#pragma unroll
    for (int k = 0; k < IPW; ++k) {
        const size_t off = min(im0 + k, d.M - 1) * L3;
        gs[k] = load3(g + off, d.N, ic);
        fp[k] = load3(F + off, d.N, ic);
    }
    const T sc = update_v ? (T)*scale : T(0);
    // |tau|^2, g.tau, l^2 of images im0 - 1 .. im1 - 1
    for (int r = im0 - 1 + wave; r < im1; r += 4) {
        double v[3];
        wave_row_sum<3>(tpart, d.nblk, r, v);
        if (lane == 0) {
            for (int q = 0; q < 3; ++q) {
                s[r - im0 + 1][q] = v[q];
                if (blockIdx.x == 0 && (r >= im0 || r == 0)) s3[r * 3 + q] = v[q];
            }
        }
    }
    __syncthreads();
    if (tid < im1 - im0) {
        const int im = im0 + tid;
        const double* s_im = s[tid + 1];
        const double inv = s_im[0] > 0.0 ? 1.0 / sqrt(s_im[0]) : 0.0;
        const int type = types[im];
        const T cpar = type == 1 ? T(2) : (type == 2 ? T(0) : T(1));
        inv_s[tid] = inv;
        gt_s[tid] = cpar * (T)(s_im[1] * inv);
        fs_s[tid] = type == 0 ? (T)(k_spring * (sqrt(s_im[2]) - sqrt(s[tid][2]))) : T(0);
        gneb_weights(E[im - 1], E[im], E[im + 1], wp_s[tid], wm_s[tid]);
    }
    __syncthreads();
    double acc[2] = {0.0, 0.0};
    double f2 = 0.0;
#pragma unroll
    for (int k = 0; k < IPW; ++k) {
        if (im0 + k < im1 && i < d.N) {
            const V3<T> n0 = xs[k + 1];
            const V3<T> t = T(inv_s[k]) * gneb_tau(xs[k], n0, xs[k + 2], wp_s[k], wm_s[k]);
            V3<T> fe = gt_s[k] * t - gs[k];
            fe = fe - dot(fe, n0) * n0;
            const V3<T> f = fe + fs_s[k] * t;
            if (update_v) {
                const V3<T> vn = sc * fp[k] + dt_2m * (fp[k] + f);
                acc[0] += (double)dot(vn, f);
            }
            store3(F + (im0 + k) * L3, d.N, i, f);
            const double ff = (double)dot(f, f);
            acc[1] += ff;
            f2 = fmax(f2, ff);
        }
    }
    block_sums<2>(acc);
    const size_t o = (size_t)blockIdx.y * d.nblk + blockIdx.x;
    if (fmax_part) {
        const double m = block_max(f2);
        if (tid == 0) fmax_part[o] = m;
    }
    if (tid == 0) {
        part[2 * o] = acc[0];
        part[2 * o + 1] = acc[1];
    }
}

// Convergence test of a chain relaxation: the largest per-spin force
// |F_{v,i}| over the interior images below tol (compared as squares).  Sets
// *stop and records the iteration that passed; later launches of the run
// see *stop and return.
__global__ void __launch_bounds__(256) k_gneb_converged(const double* __restrict__ fmax_part, int n,
                                                        double tol2, int* __restrict__ stop,
                                                        int* __restrict__ stop_iter, int iter) {
    if (*stop) return;
    double m = 0.0;
    for (int k = threadIdx.x; k < n; k += 256) m = fmax(m, fmax_part[k]);
    m = block_max(m);
    if (threadIdx.x == 0 && m < tol2) {
        *stop = 1;
        *stop_iter = iter;
    }
}

// Start of a run with a convergence test.
__global__ void k_gneb_clear_stop(int* __restrict__ stop, int* __restrict__ stop_iter) {
    if (threadIdx.x == 0) {
        *stop = 0;
        *stop_iter = -1;
    }
}

}  // namespace sp
