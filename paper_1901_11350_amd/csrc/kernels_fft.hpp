// kernels_fft.hpp -- dipole-dipole gradient by FFT convolution (Sec. III.A:
// the dipolar term as a convolution over lattice translations, with one
// interaction kernel per pair of planes).
//
// Sites i = a + Na (b + Nb p) with plane p = c + Nc beta.  The pair vector
// r_j - r_i depends on (a_j - a_i, b_j - b_i) and on the plane pair, so
//   g_i = C_dd mu_i sum_{p'} sum_{a', b'} W_{p p'}(a - a', b - b') mu_{p'} n_{p'}(a', b')
// is, for every plane pair, a 2D linear convolution with the symmetric
// tensor W = (1 - 3 r^ r^) / r^3 (W = 0 for i = j).  Zero padding to
// La >= 2 Na - 1, Lb >= 2 Nb - 1 (powers of two, at least 32) makes the
// circular convolution of the FFT equal to the linear one: only pairs inside
// the sample interact, exactly as in the direct sum.
//
// The 3P channels (component x plane) are real, so only the frequencies
// ka = 0 .. La/2 are kept.  Per evaluation three kernels:
//   k_dd_rows   two real rows (channels 2q, 2q + 1) as one complex line,
//               transformed along a and split into the two half spectra;
//   k_dd_cols   one workgroup per ka holds the columns of all channels in
//               LDS: transform along b, P x P plane-pair product with the
//               kernel spectra per frequency, transform back;
//   k_dd_out    half spectra of two channels recombined, transformed back
//               along a, scaled and written as rows of the gradient.
// Between them the half spectra lie as [ka][channel][b], so that the columns
// of one ka are contiguous; a workgroup of the row kernels takes rows side
// by side and moves them as 64-byte segments.
//
// What bounds it: on the 128x128x4 film the arrays (1.6 MB of half spectra,
// 11 MB of kernel spectra) stay in L2, and the time is launches and the
// latency of load, transform, store in each.  Eight launches with every
// transform stage between workgroup barriers and the full spectra of every
// channel passing through memory between them took 49 us per field.
#pragma once

#include "device_common.hpp"

namespace sp {

template <typename T>
struct Cx {
    T re, im;
};

template <typename T>
__device__ __forceinline__ Cx<T> cmul(Cx<T> a, Cx<T> b) {
    return Cx<T>{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}

struct FftDims {
    int Na, Nb, P;        // lattice extent along a, b; planes (Nc x basis)
    int La, Lb;           // padded transform lengths
    int Ka;               // kept frequencies along a: La / 2 + 1
    int Nc, Nbas;         // plane = c + Nc beta
};

// A line of L = 2^LOGL elements belongs to LP lanes of one wavefront, four
// elements per lane and butterfly (more butterflies per lane from 512 on),
// so the stages exchange data through LDS without a workgroup barrier.
// Lines in LDS: element e at e + e / 16 (the stride-4 stores of the first
// stages spread over the banks), PITCH apart.
template <typename T, int LOGL>
struct FftLine {
    static constexpr int L = 1 << LOGL;
    static constexpr int LP = L >= 256 ? 64 : L / 4;
    static constexpr int NB = L / 4 / LP;
    static constexpr int PITCH = L + L / 16 + 8;
    // rows of a row-kernel workgroup: 64-byte segments, at least one wavefront
    static constexpr int ROWS = 64 / (int)sizeof(Cx<T>) > 64 / LP ? 64 / (int)sizeof(Cx<T>) : 64 / LP;
    static constexpr int NT = ROWS * LP;          // its threads
};

__device__ __forceinline__ int fft_at(int e) { return e + (e >> 4); }

// Orders the LDS accesses of a wavefront's lanes: LDS serves one wavefront's
// instructions in order, so only the compiler has to be held.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Transform of one line by its LP lanes (l = lane in the line): self-sorting
// radix-4 stages (Stockham), after one radix-2 stage when LOGL is odd.  The
// first stage takes element e from ld(e), the last gives it to st(e, value);
// both walk e with neighbouring lanes on neighbouring elements.  tw: L
// twiddles exp(-2 pi i m / L).  INV: conjugated, not scaled.
template <typename T, int LOGL, bool INV, class LD, class ST>
__device__ __forceinline__ void wave_fft(Cx<T>* line, const Cx<T>* tw, int l, LD ld, ST st) {
    using F = FftLine<T, LOGL>;
    constexpr int L = F::L, LP = F::LP, NB = F::NB, H = L / 4;
    constexpr int NP = LOGL / 2;                  // radix-4 stages
    constexpr bool ODD = (LOGL & 1) != 0;
    if constexpr (ODD) {
        Cx<T> a[2 * NB], b[2 * NB];
#pragma unroll
        for (int h = 0; h < 2 * NB; ++h) {
            a[h] = ld(l + h * LP);
            b[h] = ld(l + h * LP + L / 2);
        }
        wave_sync();
#pragma unroll
        for (int h = 0; h < 2 * NB; ++h) {
            const int j = l + h * LP;
            line[fft_at(2 * j)] = Cx<T>{a[h].re + b[h].re, a[h].im + b[h].im};
            line[fft_at(2 * j + 1)] = Cx<T>{a[h].re - b[h].re, a[h].im - b[h].im};
        }
        wave_sync();
    }
#pragma unroll
    for (int s = 0; s < NP; ++s) {
        const int Ns = (ODD ? 2 : 1) << (2 * s);
        Cx<T> v[NB][4];
#pragma unroll
        for (int h = 0; h < NB; ++h) {
            const int j = l + h * LP;
            const int k = j & (Ns - 1);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = j + r * H;
                Cx<T> x;
                if (s == 0 && !ODD) x = ld(e);
                else x = line[fft_at(e)];
                if (r > 0 && Ns > 1) {
                    Cx<T> w = tw[r * k * (H / Ns)];
                    if (INV) w.im = -w.im;
                    x = cmul(x, w);
                }
                v[h][r] = x;
            }
        }
        wave_sync();
#pragma unroll
        for (int h = 0; h < NB; ++h) {
            const int j = l + h * LP;
            const int k = j & (Ns - 1);
            const int o = ((j - k) << 2) + k;
            const Cx<T> t0{v[h][0].re + v[h][2].re, v[h][0].im + v[h][2].im};
            const Cx<T> t1{v[h][0].re - v[h][2].re, v[h][0].im - v[h][2].im};
            const Cx<T> t2{v[h][1].re + v[h][3].re, v[h][1].im + v[h][3].im};
            const Cx<T> d{v[h][1].re - v[h][3].re, v[h][1].im - v[h][3].im};
            const Cx<T> t3 = INV ? Cx<T>{-d.im, d.re} : Cx<T>{d.im, -d.re};
            const Cx<T> y[4] = {{t0.re + t2.re, t0.im + t2.im}, {t1.re + t3.re, t1.im + t3.im},
                                {t0.re - t2.re, t0.im - t2.im}, {t1.re - t3.re, t1.im - t3.im}};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (s == NP - 1) st(o + r * Ns, y[r]);
                else line[fft_at(o + r * Ns)] = y[r];
            }
        }
        wave_sync();
    }
}

// Component s (xx xy xz yy yz zz) of the kernel tensor of plane-pair offset
// `off` at grid point (ia, ib), which holds the translation (da, db) =
// (a_i - a_j, b_i - b_j) with da = ia or ia - La.
// geo: A1[3], A2[3], A3[3] (Angstrom), then basis[3 * Nbas] (Angstrom).
__device__ __forceinline__ double dd_kernel_value(const FftDims& d, const double* __restrict__ geo, int off, int s,
                                                  int ia, int ib) {
    const int nb2 = d.Nbas * d.Nbas;
    const int dc = off / nb2 - (d.Nc - 1);      // c' - c
    const int beta = (off % nb2) / d.Nbas, beta2 = off % d.Nbas;
    const int da = ia < d.Na ? ia : ia - d.La;
    const int db = ib < d.Nb ? ib : ib - d.Lb;
    const bool inside = (ia < d.Na || ia > d.La - d.Na) && (ib < d.Nb || ib > d.Lb - d.Nb);
    if (!inside) return 0.0;
    // r = r_j - r_i = -da A1 - db A2 + dc A3 + basis_beta' - basis_beta
    double r[3];
    for (int k = 0; k < 3; ++k)
        r[k] = -da * geo[k] - db * geo[3 + k] + dc * geo[6 + k] + geo[9 + 3 * beta2 + k] - geo[9 + 3 * beta + k];
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    if (!(r2 > 0.0)) return 0.0;
    const double inv = 1.0 / sqrt(r2);
    const double inv3 = inv * inv * inv;
    const int p = s < 3 ? 0 : (s < 5 ? 1 : 2);
    const int q = s < 3 ? s : (s < 5 ? s - 2 : 2);
    const double e = (r[p] * inv) * (r[q] * inv);
    return ((p == q ? 1.0 : 0.0) - 3.0 * e) * inv3;
}

// Half spectra along a of the real channels 2q, 2q + 1 (q = blockIdx.y) on
// ROWS rows b.  KERNEL = false: mu_p n, channel 3p + component, Nb rows.
// KERNEL = true: the kernel tensor, channel 6 offset + component, Lb rows.
// With the complex line Z = X0 + i X1: X0^(k) = (Z^(k) + conj Z^(-k)) / 2,
// X1^(k) = (Z^(k) - conj Z^(-k)) / (2i).
template <typename T, int LOGL, bool KERNEL>
__global__ void __launch_bounds__((FftLine<T, LOGL>::NT))
    k_dd_rows(FftDims d, int channels, int rows, const T* __restrict__ n, const T* __restrict__ mu_plane,
              const double* __restrict__ geo, const Cx<T>* __restrict__ tw, Cx<T>* __restrict__ X) {
    using F = FftLine<T, LOGL>;
    constexpr int L = F::L, NT = F::NT;
    __shared__ Cx<T> buf[F::ROWS * F::PITCH];
    __shared__ Cx<T> stw[L];
    const int tid = threadIdx.x, row = tid / F::LP, l = tid % F::LP;
    const int q = blockIdx.y, b0 = blockIdx.x * F::ROWS, b = b0 + row;
    const int c0 = 2 * q, c1 = 2 * q + 1;
    for (int u = tid; u < L; u += NT) stw[u] = tw[u];
    __syncthreads();
    Cx<T>* line = buf + row * F::PITCH;
    auto put = [&](int e, Cx<T> v) { line[fft_at(e)] = v; };
    if constexpr (KERNEL) {
        auto ld = [&](int e) {
            Cx<T> z{T(0), T(0)};
            if (b < rows) {
                z.re = (T)dd_kernel_value(d, geo, c0 / 6, c0 % 6, e, b);
                if (c1 < channels) z.im = (T)dd_kernel_value(d, geo, c1 / 6, c1 % 6, e, b);
            }
            return z;
        };
        wave_fft<T, LOGL, false>(line, stw, l, ld, put);
    } else {
        const long long N = (long long)d.Na * d.Nb * d.P;
        const int p0 = c0 / 3, p1 = c1 / 3;
        const bool in = b < rows, two = c1 < channels;
        const T* x0 = n + (c0 - 3 * p0) * N + (long long)d.Na * ((in ? b : 0) + (long long)d.Nb * p0);
        const T* x1 = two ? n + (c1 - 3 * p1) * N + (long long)d.Na * ((in ? b : 0) + (long long)d.Nb * p1) : x0;
        const T m0 = mu_plane[p0], m1 = two ? mu_plane[p1] : T(0);
        auto ld = [&](int e) {
            Cx<T> z{T(0), T(0)};
            if (e < L / 2) {      // Na <= L / 2: the upper half is padding
                if (in && e < d.Na) {
                    z.re = m0 * x0[e];
                    z.im = m1 * x1[e];
                }
            }
            return z;
        };
        wave_fft<T, LOGL, false>(line, stw, l, ld, put);
    }
    __syncthreads();
    for (int u = tid; u < F::ROWS * d.Ka; u += NT) {
        const int r = u % F::ROWS, ka = u / F::ROWS;
        if (b0 + r >= rows) continue;
        const Cx<T> zk = buf[r * F::PITCH + fft_at(ka)];
        const Cx<T> zm = buf[r * F::PITCH + fft_at((L - ka) & (L - 1))];
        Cx<T>* o = X + ((long long)ka * channels + c0) * rows + b0 + r;
        o[0] = Cx<T>{T(0.5) * (zk.re + zm.re), T(0.5) * (zk.im - zm.im)};
        if (c1 < channels) o[rows] = Cx<T>{T(0.5) * (zk.im + zm.im), T(-0.5) * (zk.re - zm.re)};
    }
}

__device__ __forceinline__ constexpr int sym6(int a, int b) {
    // xx xy xz yy yz zz
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    return lo == 0 ? hi : (lo == 1 ? 2 + hi : 5);
}

// Transform along b of `lines` lines: n_in elements read (zeros beyond),
// n_out written.  In place is allowed (a line is read before it is written).
template <typename T, int LOGL, bool INV>
__global__ void __launch_bounds__(256) k_dd_lines(const Cx<T>* in, int n_in, Cx<T>* out, int n_out, long long lines,
                                                  const Cx<T>* __restrict__ tw) {
    using F = FftLine<T, LOGL>;
    constexpr int SL = 256 / F::LP;
    __shared__ Cx<T> buf[SL * F::PITCH];
    __shared__ Cx<T> stw[F::L];
    const int tid = threadIdx.x, slot = tid / F::LP, l = tid % F::LP;
    for (int u = tid; u < F::L; u += 256) stw[u] = tw[u];
    __syncthreads();
    const long long q = (long long)blockIdx.x * SL + slot;
    if (q >= lines) return;
    const Cx<T>* src = in + q * n_in;
    Cx<T>* dst = out + q * n_out;
    wave_fft<T, LOGL, INV>(
        buf + slot * F::PITCH, stw, l, [&](int e) { return e < n_in ? src[e] : Cx<T>{T(0), T(0)}; },
        [&](int e, Cx<T> v) {
            if (e < n_out) dst[e] = v;
        });
}

// Output channel spectra of one frequency:
//   G_{3p+alpha} = sum_{p', beta} W^_{p p'}^{alpha beta} X_{3p'+beta}
// W^ layout: [ka][offset][sym6][kb], offset = (c' - c + Nc - 1) Nbas^2 +
// beta Nbas + beta'.  One thread per output channel (y) and frequency.
template <typename T>
__global__ void __launch_bounds__(256) k_dd_mix(FftDims d, const Cx<T>* __restrict__ What,
                                                const Cx<T>* __restrict__ X, Cx<T>* __restrict__ G) {
    const int F = d.Ka * d.Lb, f = blockIdx.x * 256 + threadIdx.x;
    if (f >= F) return;
    const int ka = f / d.Lb, kb = f - ka * d.Lb;
    const int ch = blockIdx.y, p = ch / 3, alpha = ch - 3 * p;
    const int c = p % d.Nc, beta = p / d.Nc;
    const int C3 = 3 * d.P, noff = (2 * d.Nc - 1) * d.Nbas * d.Nbas;
    const Cx<T>* W = What + (long long)ka * noff * 6 * d.Lb + kb;
    const Cx<T>* x = X + (long long)ka * C3 * d.Lb + kb;
    Cx<T> acc{T(0), T(0)};
    for (int p2 = 0; p2 < d.P; ++p2) {
        const int c2 = p2 % d.Nc, beta2 = p2 / d.Nc;
        const int off = ((c2 - c + d.Nc - 1) * d.Nbas + beta) * d.Nbas + beta2;
#pragma unroll
        for (int bc = 0; bc < 3; ++bc) {
            const Cx<T> w = W[(long long)(off * 6 + sym6(alpha, bc)) * d.Lb];
            const Cx<T> v = x[(long long)(3 * p2 + bc) * d.Lb];
            acc.re += w.re * v.re - w.im * v.im;
            acc.im += w.re * v.im + w.im * v.re;
        }
    }
    G[((long long)ka * C3 + ch) * d.Lb + kb] = acc;
}

// Workgroup size of the fused column kernel: one (frequency, output
// component) item per thread up to Lb = 256, two or three beyond.
template <int LOGL>
constexpr int dd_cols_threads() {
    return LOGL <= 6 ? 256 : (LOGL == 7 ? 384 : (LOGL == 8 ? 768 : 1024));
}

// The columns of one ka (blockIdx.x): all 3P channels in LDS, transformed
// along b, multiplied by the kernel spectra and transformed back, Nb values
// of each channel written over the ones read.  The item (alpha, kb) forms
// component alpha of every plane; its P results stay in registers until
// every item has read the spectra.  ONE (one atom per cell): the offsets
// c' - c are walked, so each kernel value is loaded once.
template <typename T, int LOGL, int P, bool ONE>
__global__ void __launch_bounds__((dd_cols_threads<LOGL>()))
    k_dd_cols(FftDims d, const Cx<T>* __restrict__ What, Cx<T>* __restrict__ X, const Cx<T>* __restrict__ tw) {
    using F = FftLine<T, LOGL>;
    constexpr int L = F::L, NT = dd_cols_threads<LOGL>(), SL = NT / F::LP, C3 = 3 * P;
    constexpr int ITEMS = (3 * L + NT - 1) / NT;
    __shared__ Cx<T> buf[C3 * F::PITCH];
    __shared__ Cx<T> stw[L];
    const int tid = threadIdx.x, slot = tid / F::LP, l = tid % F::LP;
    const int ka = blockIdx.x;
    Cx<T>* Xk = X + (long long)ka * C3 * d.Nb;
    for (int u = tid; u < L; u += NT) stw[u] = tw[u];
    __syncthreads();
    for (int ch = slot; ch < C3; ch += SL) {
        Cx<T>* line = buf + ch * F::PITCH;
        const Cx<T>* src = Xk + ch * d.Nb;
        auto ld = [&](int e) {
            Cx<T> z{T(0), T(0)};
            if (e < L / 2) {      // Nb <= L / 2: the upper half is padding
                if (e < d.Nb) z = src[e];
            }
            return z;
        };
        wave_fft<T, LOGL, false>(line, stw, l, ld, [&](int e, Cx<T> v) { line[fft_at(e)] = v; });
    }
    __syncthreads();
    Cx<T> acc[ITEMS][P];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
#pragma unroll
        for (int p = 0; p < P; ++p) acc[it][p] = Cx<T>{T(0), T(0)};
        const int u = tid + it * NT;
        if (u >= 3 * L) continue;
        const int alpha = u >> LOGL, kb = u & (L - 1);
        const int s0 = sym6(alpha, 0), s1 = sym6(alpha, 1), s2 = sym6(alpha, 2);
        auto product = [&](const Cx<T>* w0, int p, int p2) {
            const Cx<T> w[3] = {w0[s0 * L], w0[s1 * L], w0[s2 * L]};
#pragma unroll
            for (int bc = 0; bc < 3; ++bc) {
                const Cx<T> v = buf[(3 * p2 + bc) * F::PITCH + fft_at(kb)];
                acc[it][p].re += w[bc].re * v.re - w[bc].im * v.im;
                acc[it][p].im += w[bc].re * v.im + w[bc].im * v.re;
            }
        };
        if constexpr (ONE) {
            const Cx<T>* W = What + (long long)ka * (2 * P - 1) * 6 * L + kb;
#pragma unroll
            for (int dc = 1 - P; dc < P; ++dc)
#pragma unroll
                for (int p = 0; p < P; ++p)
                    if (p + dc >= 0 && p + dc < P) product(W + (dc + P - 1) * 6 * L, p, p + dc);
        } else {
            const int noff = (2 * d.Nc - 1) * d.Nbas * d.Nbas;
            const Cx<T>* W = What + (long long)ka * noff * 6 * L + kb;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int p2 = 0; p2 < P; ++p2) {
                    const int dc = p2 % d.Nc - p % d.Nc;
                    const int off = ((dc + d.Nc - 1) * d.Nbas + p / d.Nc) * d.Nbas + p2 / d.Nc;
                    product(W + off * 6 * L, p, p2);
                }
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int u = tid + it * NT;
        if (u >= 3 * L) continue;
        const int alpha = u >> LOGL, kb = u & (L - 1);
#pragma unroll
        for (int p = 0; p < P; ++p) buf[(3 * p + alpha) * F::PITCH + fft_at(kb)] = acc[it][p];
    }
    __syncthreads();
    for (int ch = slot; ch < C3; ch += SL) {
        Cx<T>* line = buf + ch * F::PITCH;
        Cx<T>* dst = Xk + ch * d.Nb;
        auto st = [&](int e, Cx<T> v) {
            if (e < L / 2) {
                if (e < d.Nb) dst[e] = v;
            }
        };
        wave_fft<T, LOGL, true>(line, stw, l, [&](int e) { return line[fft_at(e)]; }, st);
    }
}

// Rows b of the gradient of channels 2q, 2q + 1 (q = blockIdx.y): the line
// Y = G0 + i G1 from the two half spectra (Y(-k) = conj G0(k) + i conj G1(k)),
// transformed back along a and scaled by C_dd mu_i / (La Lb).
template <typename T, int LOGL>
__global__ void __launch_bounds__((FftLine<T, LOGL>::NT))
    k_dd_out(FftDims d, const Cx<T>* __restrict__ G, const T* __restrict__ mu_plane, T scale,
             const Cx<T>* __restrict__ tw, T* __restrict__ gdd) {
    using F = FftLine<T, LOGL>;
    constexpr int L = F::L, NT = F::NT;
    __shared__ Cx<T> buf[F::ROWS * F::PITCH];
    __shared__ Cx<T> stw[L];
    const int tid = threadIdx.x, row = tid / F::LP, l = tid % F::LP;
    const int q = blockIdx.y, b0 = blockIdx.x * F::ROWS, b = b0 + row;
    const int c0 = 2 * q, c1 = 2 * q + 1, C3 = 3 * d.P;
    const bool two = c1 < C3;
    for (int u = tid; u < L; u += NT) stw[u] = tw[u];
    for (int u = tid; u < F::ROWS * d.Ka; u += NT) {
        const int r = u % F::ROWS, ka = u / F::ROWS;
        Cx<T> g0{T(0), T(0)}, g1{T(0), T(0)};
        if (b0 + r < d.Nb) {
            const Cx<T>* g = G + ((long long)ka * C3 + c0) * d.Nb + b0 + r;
            g0 = g[0];
            if (two) g1 = g[d.Nb];
        }
        if (ka > 0 && ka < L / 2)
            buf[r * F::PITCH + fft_at(L - ka)] = Cx<T>{g0.re + g1.im, g1.re - g0.im};
        buf[r * F::PITCH + fft_at(ka)] = Cx<T>{g0.re - g1.im, g0.im + g1.re};
    }
    __syncthreads();
    const long long N = (long long)d.Na * d.Nb * d.P;
    const int p0 = c0 / 3, p1 = two ? c1 / 3 : p0;
    const bool in = b < d.Nb;
    T* o0 = gdd + (c0 - 3 * p0) * N + (long long)d.Na * ((in ? b : 0) + (long long)d.Nb * p0);
    T* o1 = two ? gdd + (c1 - 3 * p1) * N + (long long)d.Na * ((in ? b : 0) + (long long)d.Nb * p1) : o0;
    const T m0 = scale * mu_plane[p0], m1 = scale * mu_plane[p1];
    Cx<T>* line = buf + row * F::PITCH;
    auto st = [&](int e, Cx<T> v) {
        if (e < L / 2) {
            if (in && e < d.Na) {
                o0[e] = m0 * v.re;
                if (two) o1[e] = m1 * v.im;
            }
        }
    };
    wave_fft<T, LOGL, true>(line, stw, l, [&](int e) { return line[fft_at(e)]; }, st);
}

}  // namespace sp
