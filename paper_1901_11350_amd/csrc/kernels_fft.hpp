// kernels_fft.hpp -- dipole-dipole gradient by FFT convolution (Sec. III.A:
// the dipolar term as a convolution over lattice translations, with one
// interaction kernel per pair of planes).
//
// Sites i = a + Na (b + Nb p) with plane p = c + Nc beta.  The pair vector
// r_j - r_i depends on (a_j - a_i, b_j - b_i) and on the plane pair, so
//   g_i = C_dd mu_i sum_{p'} sum_{a', b'} W_{p p'}(a - a', b - b') mu_{p'} n_{p'}(a', b')
// is, for every plane pair, a 2D linear convolution with the symmetric
// tensor W = (1 - 3 r^ r^) / r^3 (W = 0 for i = j).  Zero padding to
// La >= 2 Na - 1, Lb >= 2 Nb - 1 (powers of two) makes the circular
// convolution of the FFT equal to the linear one: only pairs inside the
// sample interact, exactly as in the direct sum.
//
// The 3P channels (component x plane) are real, so only the frequencies
// ka = 0 .. La/2 are kept, and two channels 2q, 2q + 1 go along a as one
// complex line, which is split into the two half spectra.  Two forms:
//   fused (up to four planes, lines of 32 points and more), half spectra as
//   [ka][b][channel]:
//     k_dd_row    one workgroup per row b, all its lines in LDS: spins to
//                 half spectra;
//     k_dd_cols   one workgroup per ka, the columns of all channels in LDS:
//                 transform along b, P x P plane-pair product with the kernel
//                 spectra per frequency, transform back;
//     k_dd_row    half spectra to rows of the gradient, or, in a step, through
//                 the step's stage to the half spectra of the new spins;
//   separate (lines of 4 points and more; an axis of one cell is not
//   transformed), half spectra as [channel][ka][b]:
//     k_dd_rows   rows of two channels, several rows side by side (64-byte
//                 segments);
//     k_dd_lines  columns, k_dd_mix the plane-pair product with one thread per
//                 channel and frequency, k_dd_lines back;
//     k_dd_out    half spectra of two channels to rows of the gradient.
//
// What bounds it: on the 128x128x4 film the arrays (1.6 MB of half spectra,
// 6.3 MB of kernel spectra) stay in L2, and the time is launches and the
// latency of load, transform, store in each.  Eight launches with every
// transform stage between workgroup barriers and the full spectra of every
// channel passing through memory between them took 49 us per field, the three
// of the fused form 17; a Depondt step 117 us, now 34.7.
#pragma once

#include "kernels_dipole.hpp"
#include "kernels_field.hpp"

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
// twiddles exp(-2 pi i m / L) in LDS.  INV: conjugated, not scaled.
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

// Plane-pair offsets are kept for dc = c' - c >= 0 only, off = (dc Nbas +
// beta) Nbas + beta': the kernel is even in r, so the spectrum of (-dc,
// beta', beta) is the conjugate of that of (dc, beta, beta').
// Component s (xx xy xz yy yz zz) of the kernel tensor of plane-pair offset
// `off` at grid point (ia, ib), which holds the translation (da, db) =
// (a_i - a_j, b_i - b_j) with da = ia or ia - La.
__device__ __forceinline__ double dd_kernel_value(const FftDims& d, const DipoleGeo& G, int off, int s, int ia,
                                                  int ib) {
    const double* geo = G.v;
    const int nb2 = d.Nbas * d.Nbas;
    const int dc = off / nb2;                   // c' - c >= 0
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
// ROWS rows b; (ka, channel, b) lies at ka ka_pitch + channel ch_pitch + b.
// KERNEL = false: mu_p n, channel 3p + component, Nb rows.
// KERNEL = true: the kernel tensor, channel 6 offset + component, Lb rows.
// With the complex line Z = X0 + i X1: X0^(k) = (Z^(k) + conj Z^(-k)) / 2,
// X1^(k) = (Z^(k) - conj Z^(-k)) / (2i).
template <typename T, int LOGL, bool KERNEL>
__global__ void __launch_bounds__((FftLine<T, LOGL>::NT))
    k_dd_rows(FftDims d, int channels, int rows, long long ka_pitch, long long ch_pitch, const T* __restrict__ n,
              const T* __restrict__ mu_plane, DipoleGeo geo, const Cx<T>* __restrict__ tw, Cx<T>* __restrict__ X) {
    using F = FftLine<T, LOGL>;
    constexpr int L = F::L, NT = F::NT;
    __shared__ Cx<T> buf[F::ROWS * F::PITCH];
    __shared__ Cx<T> wt[1 << LOGL];
    const int tid = threadIdx.x, row = tid / F::LP, l = tid % F::LP;
    const int q = blockIdx.y, b0 = blockIdx.x * F::ROWS, b = b0 + row;
    const int c0 = 2 * q, c1 = 2 * q + 1;
    for (int u = tid; u < L; u += NT) wt[u] = tw[u];
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
        wave_fft<T, LOGL, false>(line, wt, l, ld, put);
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
        wave_fft<T, LOGL, false>(line, wt, l, ld, put);
    }
    __syncthreads();
    for (int u = tid; u < F::ROWS * d.Ka; u += NT) {
        const int r = u % F::ROWS, ka = u / F::ROWS;
        if (b0 + r >= rows) continue;
        const Cx<T> zk = buf[r * F::PITCH + fft_at(ka)];
        const Cx<T> zm = buf[r * F::PITCH + fft_at((L - ka) & (L - 1))];
        Cx<T>* o = X + ka * ka_pitch + c0 * ch_pitch + b0 + r;
        o[0] = Cx<T>{T(0.5) * (zk.re + zm.re), T(0.5) * (zk.im - zm.im)};
        if (c1 < channels) o[ch_pitch] = Cx<T>{T(0.5) * (zk.im + zm.im), T(-0.5) * (zk.re - zm.re)};
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
    __shared__ Cx<T> wt[1 << LOGL];
    const int tid = threadIdx.x, slot = tid / F::LP, l = tid % F::LP;
    for (int u = tid; u < F::L; u += 256) wt[u] = tw[u];
    __syncthreads();
    const long long q = (long long)blockIdx.x * SL + slot;
    if (q >= lines) return;
    const Cx<T>* src = in + q * n_in;
    Cx<T>* dst = out + q * n_out;
    wave_fft<T, LOGL, INV>(
        buf + slot * F::PITCH, wt, l, [&](int e) { return e < n_in ? src[e] : Cx<T>{T(0), T(0)}; },
        [&](int e, Cx<T> v) {
            if (e < n_out) dst[e] = v;
        });
}

// Output channel spectra of one frequency:
//   G_{3p+alpha} = sum_{p', beta} W^_{p p'}^{alpha beta} X_{3p'+beta}
// All of them lie frequency (ka, kb) fastest, W^ as [offset][sym6][ka][kb], so
// that a wavefront reads whole lines however short the columns are.  One
// thread per output channel (y) and frequency.
template <typename T>
__global__ void __launch_bounds__(256) k_dd_mix(FftDims d, const Cx<T>* __restrict__ What,
                                                const Cx<T>* __restrict__ X, Cx<T>* __restrict__ G) {
    const int F = d.Ka * d.Lb, f = blockIdx.x * 256 + threadIdx.x;
    if (f >= F) return;
    const int ch = blockIdx.y, p = ch / 3, alpha = ch - 3 * p;
    const int c = p % d.Nc, beta = p / d.Nc;
    const Cx<T>* W = What + f;
    const Cx<T>* x = X + f;
    Cx<T> acc{T(0), T(0)};
    for (int p2 = 0; p2 < d.P; ++p2) {
        const int dc = p2 % d.Nc - c, beta2 = p2 / d.Nc;
        const int off = dc >= 0 ? (dc * d.Nbas + beta) * d.Nbas + beta2 : (-dc * d.Nbas + beta2) * d.Nbas + beta;
        const T sign = dc >= 0 ? T(1) : T(-1);
#pragma unroll
        for (int bc = 0; bc < 3; ++bc) {
            Cx<T> w = W[(long long)(off * 6 + sym6(alpha, bc)) * F];
            w.im *= sign;
            const Cx<T> v = x[(long long)(3 * p2 + bc) * F];
            acc.re += w.re * v.re - w.im * v.im;
            acc.im += w.re * v.im + w.im * v.re;
        }
    }
    G[(long long)ch * F + f] = acc;
}

// Workgroup size of the fused column kernel: one (frequency, output
// component) item per thread up to Lb = 256 (twelve wavefronts, one per
// channel of four planes), two or three beyond.
template <int LOGL>
constexpr int dd_cols_threads() {
    return LOGL <= 6 ? 256 : (LOGL == 7 ? 384 : (LOGL == 8 ? 768 : 1024));
}

// The columns of one ka (blockIdx.x) of X [ka][b][channel]: all 3P channels
// in LDS, transformed along b, multiplied by the kernel spectra and
// transformed back, Nb values of each channel written over the ones read.
// The item (alpha, kb) forms component alpha of every plane; its P results
// stay in registers until every item has read the spectra.  ONE (one atom
// per cell): the offsets c' - c are walked, so each kernel value is loaded
// once and serves +dc and, conjugated, -dc; with one item per thread the
// loads are issued before the transform, whose time hides them.
template <typename T, int LOGL, int P, bool ONE>
__global__ void __launch_bounds__((dd_cols_threads<LOGL>()))
    k_dd_cols(FftDims d, const Cx<T>* __restrict__ What, Cx<T>* __restrict__ X, const Cx<T>* __restrict__ tw) {
    using F = FftLine<T, LOGL>;
    constexpr int L = F::L, NT = dd_cols_threads<LOGL>(), SL = NT / F::LP, C3 = 3 * P;
    constexpr int ITEMS = (3 * L + NT - 1) / NT;
    constexpr bool PRE = ONE && ITEMS == 1;
    __shared__ Cx<T> buf[C3 * F::PITCH];
    __shared__ Cx<T> wt[1 << LOGL];
    const int tid = threadIdx.x, slot = tid / F::LP, l = tid % F::LP;
    const int ka = blockIdx.x;
    Cx<T>* Xk = X + (long long)ka * C3 * d.Nb;
    constexpr int XR = (C3 * L / 2 + NT - 1) / NT;     // rounds of the staging load
    Cx<T> x0[XR];
#pragma unroll
    for (int k = 0; k < XR; ++k)
        if (tid + k * NT < C3 * d.Nb) x0[k] = Xk[tid + k * NT];
    Cx<T> t0{T(0), T(0)};
    if (tid < L) t0 = tw[tid];
    const int noff = ONE ? P : d.Nc * d.Nbas * d.Nbas;
    const Cx<T>* W = What + (long long)ka * noff * 6 * L;
    Cx<T> wpre[PRE ? P : 1][3];
    if constexpr (PRE) {
        if (tid < 3 * L) {
            const int alpha = tid >> LOGL;
#pragma unroll
            for (int o = 0; o < P; ++o)
#pragma unroll
                for (int bc = 0; bc < 3; ++bc) wpre[o][bc] = W[(o * 6 + sym6(alpha, bc)) * L + (tid & (L - 1))];
        }
    }
#pragma unroll
    for (int k = 0; k < XR; ++k) {
        const int u = tid + k * NT;
        const int b = u / C3, ch = u - b * C3;
        if (u < C3 * d.Nb) buf[ch * F::PITCH + fft_at(b)] = x0[k];
    }
    if (tid < L) wt[tid] = t0;
    for (int u = tid + NT; u < L; u += NT) wt[u] = tw[u];
    __syncthreads();
    for (int ch = slot; ch < C3; ch += SL) {
        Cx<T>* line = buf + ch * F::PITCH;
        auto ld = [&](int e) {
            Cx<T> z{T(0), T(0)};
            if (e < L / 2) {      // Nb <= L / 2: the upper half is padding
                if (e < d.Nb) z = line[fft_at(e)];
            }
            return z;
        };
        wave_fft<T, LOGL, false>(line, wt, l, ld, [&](int e, Cx<T> v) { line[fft_at(e)] = v; });
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
        // component alpha of plane p += w (conjugated: w*) times the spins of plane p2
        auto product = [&](const Cx<T>* w, bool conjugate, int p, int p2) {
#pragma unroll
            for (int bc = 0; bc < 3; ++bc) {
                const Cx<T> v = buf[(3 * p2 + bc) * F::PITCH + fft_at(kb)];
                const T im = conjugate ? -w[bc].im : w[bc].im;
                acc[it][p].re += w[bc].re * v.re - im * v.im;
                acc[it][p].im += w[bc].re * v.im + im * v.re;
            }
        };
        if constexpr (ONE) {
#pragma unroll
            for (int dc = 0; dc < P; ++dc) {
                Cx<T> w[3];
                if constexpr (PRE) {
#pragma unroll
                    for (int bc = 0; bc < 3; ++bc) w[bc] = wpre[dc][bc];
                } else {
                    const Cx<T>* w0 = W + dc * 6 * L + kb;
                    w[0] = w0[s0 * L];
                    w[1] = w0[s1 * L];
                    w[2] = w0[s2 * L];
                }
#pragma unroll
                for (int p = 0; p + dc < P; ++p) {
                    product(w, false, p, p + dc);
                    if (dc > 0) product(w, true, p + dc, p);
                }
            }
        } else {
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int p2 = 0; p2 < P; ++p2) {
                    const int dc = p2 % d.Nc - p % d.Nc, beta = p / d.Nc, beta2 = p2 / d.Nc;
                    const int off = dc >= 0 ? (dc * d.Nbas + beta) * d.Nbas + beta2
                                            : (-dc * d.Nbas + beta2) * d.Nbas + beta;
                    const Cx<T>* w0 = W + off * 6 * L + kb;
                    const Cx<T> w[3] = {w0[s0 * L], w0[s1 * L], w0[s2 * L]};
                    product(w, dc < 0, p, p2);
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
        auto st = [&](int e, Cx<T> v) {
            if (e < L / 2) line[fft_at(e)] = v;
        };
        wave_fft<T, LOGL, true>(line, wt, l, [&](int e) { return line[fft_at(e)]; }, st);
    }
    __syncthreads();
    for (int u = tid; u < C3 * d.Nb; u += NT) {
        const int b = u / C3, ch = u - b * C3;
        Xk[u] = buf[ch * F::PITCH + fft_at(b)];
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
    __shared__ Cx<T> wt[1 << LOGL];
    const int tid = threadIdx.x, row = tid / F::LP, l = tid % F::LP;
    const int q = blockIdx.y, b0 = blockIdx.x * F::ROWS, b = b0 + row;
    const int c0 = 2 * q, c1 = 2 * q + 1, C3 = 3 * d.P;
    const bool two = c1 < C3;
    for (int u = tid; u < L; u += NT) wt[u] = tw[u];
    for (int u = tid; u < F::ROWS * d.Ka; u += NT) {
        const int r = u % F::ROWS, ka = u / F::ROWS;
        Cx<T> g0{T(0), T(0)}, g1{T(0), T(0)};
        if (b0 + r < d.Nb) {
            const Cx<T>* g = G + ((long long)c0 * d.Ka + ka) * d.Nb + b0 + r;
            g0 = g[0];
            if (two) g1 = g[(long long)d.Ka * d.Nb];
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
    wave_fft<T, LOGL, true>(line, wt, l, [&](int e) { return line[fft_at(e)]; }, st);
}

// ------------------------------------------- row kernel of the fused form
// One workgroup per row b holds the lines of all 3P <= 12 channels of that
// row in LDS (two channels per complex line, one wavefront per line while it
// is transformed), so the whole chain of a half step from the dipole spectra
// to the spectra of the new spins stays in it:
//   DD_SPECTRA   spins -> half spectra
//   DD_FIELD     half spectra of the field -> gdd
//   DD_PREDICT   half spectra of the field -> predictor step -> half spectra
//   DD_CORRECT   the same with the corrector
// The half spectra X [ka][b][channel] are read and written by the row's own
// workgroup only (in place).  The local field of a thread's first site is
// formed while the spectra are on their way.  A site's gradient component
// sits in the float of its channel's line and is replaced there by the new
// spin component by the thread that read it.
enum DdStage { DD_SPECTRA = 0, DD_FIELD = 1, DD_PREDICT = 2, DD_CORRECT = 3 };
constexpr int kDdRowThreads = 512;
constexpr int kDdMaxPlanes = 4;

__device__ __forceinline__ int lane_value(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float lane_value(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Local gradient terms of site (a, row b, plane c, atom beta): site_terms
// with everything but `a` uniform over the wavefront.  Lane q prepares bond
// q (its record, the wraps along b and c, the first site of the partner's
// row; zero couplings where the row lies outside the sample or the bond
// comes back to its own site), 64 bonds at a time, and the prepared values
// go to scalar registers lane by lane; the neighbours of four bonds are in
// flight together.
template <typename T>
__device__ __forceinline__ V3<T> row_gradient(const Lattice& L, const BondCoef<T>& C, const Phys<T>& P,
                                              const T* __restrict__ n, int a, int b, int c, int beta, V3<T> ni) {
    const int na = L.n[0], nb = L.n[1], nc = L.n[2], N = L.N;
    const char* nx = reinterpret_cast<const char*>(n);
    const char* ny = reinterpret_cast<const char*>(n + N);
    const char* nz = reinterpret_cast<const char*>(n + 2 * (size_t)N);
    const int lane = threadIdx.x & 63;
    const int self = na * (b + nb * (c + nc * beta));
    V3<T> gj{T(0), T(0), T(0)}, gd{T(0), T(0), T(0)};
    const int q1 = L.bstart[beta + 1];
    for (int q0 = L.bstart[beta]; q0 < q1; q0 += 64) {
        const int cnt = min(64, q1 - q0);
        int base = self, da = 0;
        T rJ = T(0), rD[3] = {T(0), T(0), T(0)};
        if (lane < cnt) {
            const int4 rec = L.bond[q0 + lane];
            const T J = C.J[q0 + lane];
            const V3<T> D{C.D[3 * (q0 + lane)], C.D[3 * (q0 + lane) + 1], C.D[3 * (q0 + lane) + 2]};
            bool ok = true;
            const int tb = wrap_coord(b + rec.z, nb, L.per[1], ok);
            const int tc = wrap_coord(c + rec.w, nc, L.per[2], ok);
            int d = rec.y;
            if (L.per[0]) {             // 0 .. na - 1: one wrap reaches the partner
                d %= na;
                d += d < 0 ? na : 0;
            }
            const int row = na * (tb + nb * (tc + nc * rec.x));
            if (ok && !(row == self && d == 0)) {
                base = row;
                da = d;
                rJ = J;
                rD[0] = D.x;
                rD[1] = D.y;
                rD[2] = D.z;
            }
        }
        const bool dmi = __ballot(rD[0] != T(0) || rD[1] != T(0) || rD[2] != T(0)) != 0;
        for (int u0 = 0; u0 < cnt; u0 += 4) {
            V3<T> nj[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                int ta = a + lane_value(da, u0 + u);
                bool in = true;
                if (L.per[0]) ta -= ta >= na ? na : 0;
                else in = (unsigned)ta < (unsigned)na;
                const uint32_t off = (uint32_t)(lane_value(base, u0 + u) + (in ? ta : 0)) * (uint32_t)sizeof(T);
                const V3<T> v{*reinterpret_cast<const T*>(nx + off), *reinterpret_cast<const T*>(ny + off),
                              *reinterpret_cast<const T*>(nz + off)};
                nj[u] = V3<T>{in ? v.x : T(0), in ? v.y : T(0), in ? v.z : T(0)};
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                gj = gj - lane_value(rJ, u0 + u) * nj[u];
                if (dmi)
                    gd = gd - cross(nj[u], V3<T>{lane_value(rD[0], u0 + u), lane_value(rD[1], u0 + u),
                                                 lane_value(rD[2], u0 + u)});
            }
        }
    }
    FieldTerms<T> f;
    f.z = V3<T>{P.gZ[beta][0], P.gZ[beta][1], P.gZ[beta][2]};
    const V3<T> ax{P.Kax[beta][0], P.Kax[beta][1], P.Kax[beta][2]};
    f.k = (-P.K2[beta] * dot(ax, ni)) * ax;
    f.q = gauss_gradient(P, ni);
    f.j = gj;
    f.d = gd;
    return total(f);
}

template <typename T, int LOGL, int STAGE>
__global__ void __launch_bounds__(kDdRowThreads)
    k_dd_row(FftDims d, Lattice L, BondCoef<T> C, Phys<T> P, LLGArgs<T> A_arg, int solver,
             const int* __restrict__ abort_flag, const T* __restrict__ mu_plane, T scale,
             const Cx<T>* __restrict__ tw, Cx<T>* X, const T* __restrict__ m, const T* __restrict__ n,
             T* __restrict__ Abuf, T* __restrict__ out) {
    // a stopped run still computes, and stores nothing
    const int stop = STAGE >= DD_PREDICT && abort_flag ? *abort_flag : 0;
    using F = FftLine<T, LOGL>;
    constexpr int LL = F::L, Q = (3 * kDdMaxPlanes + 1) / 2;
    __shared__ Cx<T> buf[Q * F::PITCH];
    __shared__ Cx<T> wt[1 << LOGL];
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int b = blockIdx.x;
    const int C3 = 3 * d.P, nq = (C3 + 1) / 2, N = L.N;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = nthr >> 6, lane = tid & 63;
    const int segs = (d.Na + 63) / 64, items = segs * d.P;
    Cx<T>* Xb = X + (long long)b * C3;
    const long long ka_pitch = (long long)d.Nb * C3;
    T* slots = reinterpret_cast<T*>(buf);
    auto slot = [&](int ch, int a) -> T& { return slots[((ch >> 1) * F::PITCH + fft_at(a)) * 2 + (ch & 1)]; };
    LLGArgs<T> A = A_arg;
    if constexpr (STAGE >= DD_PREDICT) A = resolve_step(A_arg);

    // field spectra -> lines Y = G0 + i G1: the first GU rounds of loads are
    // issued here and stored after the local field
    constexpr int GU = STAGE == DD_SPECTRA ? 1 : 4;
    Cx<T> g0[GU], g1[GU];
    auto get = [&](int u, Cx<T>& x, Cx<T>& y) {
        const int ka = u / nq, q = u - ka * nq;
        const Cx<T>* g = Xb + ka * ka_pitch + 2 * q;
        x = g[0];
        y = 2 * q + 1 < C3 ? g[1] : Cx<T>{T(0), T(0)};
    };
    auto put = [&](int u, Cx<T> x, Cx<T> y) {
        const int ka = u / nq, q = u - ka * nq;
        Cx<T>* line = buf + q * F::PITCH;
        if (ka > 0 && ka < LL / 2) line[fft_at(LL - ka)] = Cx<T>{x.re + y.im, y.re - x.im};
        line[fft_at(ka)] = Cx<T>{x.re - y.im, x.im + y.re};
    };
    if constexpr (STAGE != DD_SPECTRA) {
#pragma unroll
        for (int k = 0; k < GU; ++k)
            if (tid + k * nthr < d.Ka * nq) get(tid + k * nthr, g0[k], g1[k]);
    }
    const int lw = tid / F::LP, l = tid % F::LP;   // line slots: LP lanes each
    const int nslots = nthr / F::LP;
    Cx<T> t0{T(0), T(0)};
    if (tid < LL) t0 = tw[tid];

    // m: the spins whose dipole field the spectra hold (n, or the predictor's)
    struct Site {
        int i, beta;
        V3<T> m, g;
    };
    auto local = [&](int it) {
        const int p = it / segs, a = (it - p * segs) * 64 + lane;
        Site t;
        const int c = p % d.Nc;
        t.beta = p / d.Nc;
        const int ac = min(a, d.Na - 1);
        t.i = ac + d.Na * (b + d.Nb * p);
        t.m = load3(m, N, t.i);
        t.g = V3<T>{T(0), T(0), T(0)};
        if constexpr (STAGE >= DD_PREDICT) t.g = row_gradient(L, C, P, m, ac, b, c, t.beta, t.m);
        return t;
    };
    auto finish = [&](int it, const Site& s) {
        const int p = it / segs, a = (it - p * segs) * 64 + lane;
        if (a >= d.Na) return;
        V3<T> o = s.m;
        if constexpr (STAGE != DD_SPECTRA) {
            const T sc = scale * mu_plane[p];
            const V3<T> dip{sc * slot(3 * p, a), sc * slot(3 * p + 1, a), sc * slot(3 * p + 2, a)};
            if constexpr (STAGE == DD_FIELD) {
                store3(out, N, s.i, dip);
                return;
            } else {
                const V3<T> g = s.g + dip;
                const T inv_m = T(1) / P.mumuB[s.beta];
                V3<T> B = (-inv_m) * g;
                if (A.thermal) B = B + P.sigma[s.beta] * normals3(thermal_bits(A.key, (uint32_t)s.i), T(0));
                const V3<T> Ai = llg_A(s.m, B, A.gp, A.alpha);
                if constexpr (STAGE == DD_PREDICT) {
                    if (solver == SOLVER_HEUN) {
                        const V3<T> f = cross(s.m, Ai);
                        store3(Abuf, N, s.i, f);
                        o = normalize3(s.m + A.dt * f);
                    } else if (solver == SOLVER_SIB) {
                        o = T(0.5) * (s.m + sib_stage(s.m, Ai, A.dt));
                    } else {
                        store3(Abuf, N, s.i, Ai);
                        o = renorm_if_float(rotate(s.m, T(-1) * Ai, A.dt));
                    }
                } else {
                    const V3<T> ni = load3(n, N, s.i);
                    if (solver == SOLVER_HEUN) {
                        const V3<T> f0 = load3(Abuf, N, s.i);
                        o = normalize3(ni + (T(0.5) * A.dt) * (f0 + cross(s.m, Ai)));
                    } else if (solver == SOLVER_SIB) {
                        o = renorm_if_float(sib_stage(ni, Ai, A.dt));
                    } else {
                        const V3<T> A0 = load3(Abuf, N, s.i);
                        o = renorm_if_float(rotate(ni, T(-0.5) * (A0 + Ai), A.dt));
                    }
                }
                store3(out, N, s.i, o);
            }
        }
        const T mu = mu_plane[p];
        slot(3 * p, a) = mu * o.x;
        slot(3 * p + 1, a) = mu * o.y;
        slot(3 * p + 2, a) = mu * o.z;
    };
    Site first{};
    if (wave < items) first = local(wave);
    if constexpr (STAGE != DD_SPECTRA) {
#pragma unroll
        for (int k = 0; k < GU; ++k)
            if (tid + k * nthr < d.Ka * nq) put(tid + k * nthr, g0[k], g1[k]);
        for (int u = tid + GU * nthr; u < d.Ka * nq; u += nthr) {
            get(u, g0[0], g1[0]);
            put(u, g0[0], g1[0]);
        }
    }
    if (tid < LL) wt[tid] = t0;
    for (int u = tid + nthr; u < LL; u += nthr) wt[u] = tw[u];
    __syncthreads();
    if constexpr (STAGE != DD_SPECTRA) {
        for (int q = lw; q < nq; q += nslots) {
            Cx<T>* line = buf + q * F::PITCH;
            auto st = [&](int e, Cx<T> v) {
                if (e < LL / 2) line[fft_at(e)] = v;
            };
            wave_fft<T, LOGL, true>(line, wt, l, [&](int e) { return line[fft_at(e)]; }, st);
        }
        __syncthreads();
    }
    if (stop) return;
    if (wave < items) finish(wave, first);
    for (int it = wave + waves; it < items; it += waves) finish(it, local(it));
    if constexpr (STAGE == DD_FIELD) return;
    __syncthreads();
    for (int q = lw; q < nq; q += nslots) {
        Cx<T>* line = buf + q * F::PITCH;
        const bool two = 2 * q + 1 < C3;
        auto ld = [&](int e) {
            Cx<T> z{T(0), T(0)};
            if (e < LL / 2) {      // Na <= L / 2: the upper half is padding
                if (e < d.Na) {
                    z = line[fft_at(e)];
                    if (!two) z.im = T(0);
                }
            }
            return z;
        };
        wave_fft<T, LOGL, false>(line, wt, l, ld, [&](int e, Cx<T> v) { line[fft_at(e)] = v; });
    }
    __syncthreads();
    for (int u = tid; u < d.Ka * nq; u += nthr) {
        const int ka = u / nq, q = u - ka * nq;
        const Cx<T>* line = buf + q * F::PITCH;
        const Cx<T> zk = line[fft_at(ka)];
        const Cx<T> zm = line[fft_at((LL - ka) & (LL - 1))];
        Cx<T>* o = Xb + ka * ka_pitch + 2 * q;
        o[0] = Cx<T>{T(0.5) * (zk.re + zm.re), T(0.5) * (zk.im - zm.im)};
        if (2 * q + 1 < C3) o[1] = Cx<T>{T(0.5) * (zk.im + zm.im), T(-0.5) * (zk.re - zm.re)};
    }
}

}  // namespace sp
