// kernels_fused2d.hpp -- fused Depondt step for one-atom 2D lattices with a
// compile-time neighbour stencil.
//
// A stencil "shape" is the list of cell offsets (da, db) of the bonds of one
// site, grouped by neighbour shell; the host matches the bond table against
// the shapes below and passes the per-shell exchange constants and per-bond
// DMI vectors at run time.  With the offsets known at compile time the LDS
// neighbour reads use immediate offsets, exchange is summed per shell before
// multiplying by J, and (bonds being in-plane) every DMI vector has D_z = 0,
// so n_j x D costs four FMAs.
//
// Per workgroup (NT threads, TX x TY output tile):
//   1. stage n(t) on the tile plus a 2R halo into LDS, one 16-byte cell per
//      site (periodic axes wrap, open axes pad with zero spins, which drop
//      out of every bond sum); the external plus thermal field of the cells
//      a thread will predict (Philox, counter = global site) is formed while
//      these loads are in flight;
//   2. predictor on the tile plus an R halo: field B in Tesla (coefficients
//      divided by mu mu_B on the host), w = B + alpha n x B (A = -gp w),
//      n^p = R(A) n into LDS; w and the base field of the tile sites stay in
//      the registers of the thread that owns the site;
//   3. corrector on the tile: w^p from n^p, n(t+dt) = R((A + A^p)/2) n(t),
//      written once to HBM.
// Workgroups are mapped to tiles so that each XCD (workgroups are dealt to
// the 8 XCDs round-robin) owns a contiguous band of tile rows: neighbouring
// tiles, whose halos overlap, then share one L2.
#pragma once

#include "kernels_field.hpp"

namespace sp {

enum Shape2D { SH_SQ1 = 0, SH_SQ2, SH_SQ3, SH_TRI1, SH_TRI2, SH_TRI3, SH_COUNT };

template <int S>
struct ShapeTab;

// square lattice: shells at 1, sqrt2, 2
template <>
struct ShapeTab<SH_SQ1> {
    static constexpr int NB = 4, NS = 1, R = 1, NB0 = 4;
    static constexpr int da[NB] = {1, -1, 0, 0};
    static constexpr int db[NB] = {0, 0, 1, -1};
    static constexpr int sh[NB] = {0, 0, 0, 0};
};
template <>
struct ShapeTab<SH_SQ2> {
    static constexpr int NB = 8, NS = 2, R = 1, NB0 = 4;
    static constexpr int da[NB] = {1, -1, 0, 0, 1, -1, 1, -1};
    static constexpr int db[NB] = {0, 0, 1, -1, 1, -1, -1, 1};
    static constexpr int sh[NB] = {0, 0, 0, 0, 1, 1, 1, 1};
};
template <>
struct ShapeTab<SH_SQ3> {
    static constexpr int NB = 12, NS = 3, R = 2, NB0 = 4;
    static constexpr int da[NB] = {1, -1, 0, 0, 1, -1, 1, -1, 2, -2, 0, 0};
    static constexpr int db[NB] = {0, 0, 1, -1, 1, -1, -1, 1, 0, 0, 2, -2};
    static constexpr int sh[NB] = {0, 0, 0, 0, 1, 1, 1, 1, 2, 2, 2, 2};
};
// triangular lattice a1 = (1,0), a2 = (1/2, sqrt3/2): shells at 1, sqrt3, 2
template <>
struct ShapeTab<SH_TRI1> {
    static constexpr int NB = 6, NS = 1, R = 1, NB0 = 6;
    static constexpr int da[NB] = {1, -1, 0, 0, 1, -1};
    static constexpr int db[NB] = {0, 0, 1, -1, -1, 1};
    static constexpr int sh[NB] = {0, 0, 0, 0, 0, 0};
};
template <>
struct ShapeTab<SH_TRI2> {
    static constexpr int NB = 12, NS = 2, R = 2, NB0 = 6;
    static constexpr int da[NB] = {1, -1, 0, 0, 1, -1, 1, -1, 2, -2, 1, -1};
    static constexpr int db[NB] = {0, 0, 1, -1, -1, 1, 1, -1, -1, 1, -2, 2};
    static constexpr int sh[NB] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1};
};
template <>
struct ShapeTab<SH_TRI3> {
    static constexpr int NB = 18, NS = 3, R = 2, NB0 = 6;
    static constexpr int da[NB] = {1, -1, 0, 0, 1, -1, 1, -1, 2, -2, 1, -1, 2, -2, 0, 0, 2, -2};
    static constexpr int db[NB] = {0, 0, 1, -1, -1, 1, 1, -1, -1, 1, -2, 2, 0, 0, 2, -2, -2, 2};
    static constexpr int sh[NB] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 2, 2, 2, 2, 2, 2};
};

// Run-time coefficients in shape order.
template <typename T>
struct ShapeCoef {
    T J[4];            // per shell
    T Dx[24], Dy[24];  // per bond (D_z = 0 for in-plane bonds)
};

// The same divided by mu mu_B, for the step kernels: their bond sums then
// give the field B = -dH/dn / (mu mu_B) in Tesla directly, starting from
// the external (plus thermal) field.
template <typename T>
struct StepCoef {
    T J[4];
    T Dx[24], Dy[24];
    T K2;        // 2K / (mu mu_B)
    T Bext[3];   // external field (Tesla)
};

template <typename T>
__device__ __forceinline__ void native_sincos(T x, T* s, T* c) {
    if constexpr (sizeof(T) == 4) {
        const float r = x * 0.15915494309189535f;  // radians -> revolutions
        *s = __builtin_amdgcn_sinf(r);
        *c = __builtin_amdgcn_cosf(r);
    } else {
        sincos(x, s, c);
    }
}

// LLG rotation vector without its prefactor: with w = B + alpha n x B the
// equation dn/dt = n x A, A = -gp w, reads dn/dt = gp w x n, so a step
// turns n about w by gp |w| dt (Depondt's scheme, Appendix B).
template <typename T>
__device__ __forceinline__ V3<T> llg_w(V3<T> n, V3<T> B, T alpha) {
    const V3<T> nxB = cross(n, B);
    return V3<T>{B.x + alpha * nxB.x, B.y + alpha * nxB.y, B.z + alpha * nxB.z};
}

// Half-angle factor h of rotate_half for a turn by gp |w| dt: gp dt / 2, in
// revolutions for FP32 (the unit of the hardware sine and cosine), radians
// for FP64.
template <typename T>
__device__ __forceinline__ T rot_half_factor(T gp, T dt) {
    if constexpr (sizeof(T) == 4) {
        return (0.5f * 0.15915494309189535f) * (gp * dt);
    } else {
        return T(0.5) * (gp * dt);
    }
}

// Rotation of n about w by the angle theta = 2 h |w|, in the form
//   n' = n + s1 (w x n) + s2 (w (w.n) - |w|^2 n),
//   s1 = sin(theta)/|w|, s2 = (1 - cos theta)/|w|^2 = 2 sin^2(theta/2)/|w|^2.
// w = 0 leaves n unchanged: in FP32 the 1e-30 added to |w|^2 keeps 1/|w|
// finite and is below the rounding of any |w|^2 above 3e-23.
template <typename T>
__device__ __forceinline__ V3<T> rotate_half(V3<T> n, V3<T> w, T h) {
    const T w2 = dot(w, w);
    T inv, sh, ch;
    if constexpr (sizeof(T) == 4) {
        inv = __builtin_amdgcn_rsqf(w2 + 1e-30f);
        const float half = h * (w2 * inv);
        sh = __builtin_amdgcn_sinf(half);
        ch = __builtin_amdgcn_cosf(half);
    } else {
        inv = w2 > 0.0 ? 1.0 / sqrt(w2) : 0.0;
        sincos(h * (w2 * inv), &sh, &ch);
    }
    // t = sin(theta/2) / |w|: s1 = 2 t cos(theta/2), s2 = 2 t^2
    const T t = sh * inv;
    const T t2 = t + t;
    const T s1 = t2 * ch;
    const T s2 = t2 * t;
    const V3<T> wxn = cross(w, n);
    const T wn = dot(w, n);
    return V3<T>{n.x + s1 * wxn.x + s2 * (w.x * wn - w2 * n.x),
                 n.y + s1 * wxn.y + s2 * (w.y * wn - w2 * n.y),
                 n.z + s1 * wxn.z + s2 * (w.z * wn - w2 * n.z)};
}

// Site spin padded to 16 (FP32) or 32 (FP64) bytes, so that one LDS read
// with an immediate offset fetches a neighbour.
template <typename T>
struct alignas(4 * sizeof(T)) V4 {
    T x, y, z, w;
};

// Store of a kernel's output spin or field.  An agent-scope store is written
// through to the device coherence point instead of staying dirty in the
// writing XCD's L2, so the L2 write-back that ends the kernel (it makes the
// output visible to the next launch on every XCD) finds little to do.
// Semantically a plain store: the kernel boundary orders it.
template <typename T>
__device__ __forceinline__ void store_out(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One FP32 LDS cell read as a whole 16-byte ds_read_b128.  Left to itself
// the compiler drops the unused padding word and emits ds_read_b96, which
// on gfx950 costs ~8.7 LDS cycles per wave against ~4.9 for b128 (a wave of
// 16-byte-strided cells); the empty asm keeps the fourth word live, so the
// full-width read is kept, at no arithmetic cost.
template <typename T>
__device__ __forceinline__ V3<T> lds_cell_xyz(const V4<T>* __restrict__ sv, int o) {
    const V4<T> v = sv[o];
    if constexpr (sizeof(T) == 4) asm volatile("" ::"v"(v.w));
    return V3<T>{v.x, v.y, v.z};
}

// True when bond q is the first of its shell in the stencil's order (folds
// to a constant once a bond loop is unrolled).
template <typename SH>
__device__ constexpr bool first_of_shell(int q) {
    for (int r = 0; r < q; ++r)
        if (SH::sh[r] == SH::sh[q]) return false;
    return true;
}

// shape_field on 16-byte LDS cells: neighbours are read six at a time, with
// one empty asm after each group keeping the padding words live, so a
// group's reads are in flight together (one wait per group instead of one
// per read); shell sums start from their first neighbour.
template <typename T, int S, int NDMI, int W>
__device__ __forceinline__ V3<T> shape_field_aos(const ShapeCoef<T>& C, const Site2D<T>& Q,
                                                 const V4<T>* __restrict__ sv, int c, V3<T> ni) {
    using SH = ShapeTab<S>;
    constexpr int G = 6;
    V3<T> acc[SH::NS];
    T dx = T(0), dy = T(0), dz = T(0);
#pragma unroll
    for (int q0 = 0; q0 < SH::NB; q0 += G) {
        V4<T> v[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int q = q0 + k;
            if (q < SH::NB)
                v[k] = sv[c + SH::da[q] + SH::db[q] * W];
            else
                v[k] = v[0];
        }
        if constexpr (sizeof(T) == 4)
            asm volatile("" ::"v"(v[0].w), "v"(v[1].w), "v"(v[2].w), "v"(v[3].w), "v"(v[4].w), "v"(v[5].w));
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int q = q0 + k;
            if (q < SH::NB) {
                const V3<T> nj{v[k].x, v[k].y, v[k].z};
                const int sh = SH::sh[q];
                if (first_of_shell<SH>(q)) {
                    acc[sh] = nj;
                } else {
                    acc[sh].x += nj.x;
                    acc[sh].y += nj.y;
                    acc[sh].z += nj.z;
                }
                if (q < NDMI) {
                    // n_j x D with D = (Dx, Dy, 0)
                    dx -= nj.z * C.Dy[q];
                    dy += nj.z * C.Dx[q];
                    dz += nj.x * C.Dy[q] - nj.y * C.Dx[q];
                }
            }
        }
    }
    const T kn = Q.K2 * (Q.Kax[0] * ni.x + Q.Kax[1] * ni.y + Q.Kax[2] * ni.z);
    V3<T> g{Q.gZ[0] - kn * Q.Kax[0] - dx, Q.gZ[1] - kn * Q.Kax[1] - dy, Q.gZ[2] - kn * Q.Kax[2] - dz};
#pragma unroll
    for (int s = 0; s < SH::NS; ++s) {
        g.x -= C.J[s] * acc[s].x;
        g.y -= C.J[s] * acc[s].y;
        g.z -= C.J[s] * acc[s].z;
    }
    return g;
}

// The field B (Tesla) of a step kernel on 16-byte LDS cells, read as in
// shape_field_aos, from coefficients divided by mu mu_B and starting from
// base (external plus thermal field): each coefficient (a scalar register)
// enters one multiply-add per component.
template <typename T, int S, int NDMI, int W>
__device__ __forceinline__ V3<T> shape_B_aos(const StepCoef<T>& C, const Site2D<T>& Q, const V4<T>* __restrict__ sv,
                                             int c, V3<T> ni, V3<T> base) {
    using SH = ShapeTab<S>;
    constexpr int G = 6;
    V3<T> acc[SH::NS];
    V3<T> B = base;
#pragma unroll
    for (int q0 = 0; q0 < SH::NB; q0 += G) {
        V4<T> v[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int q = q0 + k;
            if (q < SH::NB)
                v[k] = sv[c + SH::da[q] + SH::db[q] * W];
            else
                v[k] = v[0];
        }
        if constexpr (sizeof(T) == 4)
            asm volatile("" ::"v"(v[0].w), "v"(v[1].w), "v"(v[2].w), "v"(v[3].w), "v"(v[4].w), "v"(v[5].w));
#pragma unroll
        for (int k = 0; k < G; ++k) {
            const int q = q0 + k;
            if (q < SH::NB) {
                const V3<T> nj{v[k].x, v[k].y, v[k].z};
                const int sh = SH::sh[q];
                if (first_of_shell<SH>(q)) {
                    acc[sh] = nj;
                } else {
                    acc[sh].x += nj.x;
                    acc[sh].y += nj.y;
                    acc[sh].z += nj.z;
                }
                if (q < NDMI) {
                    // + n_j x D with D = (Dx, Dy, 0)
                    B.x -= nj.z * C.Dy[q];
                    B.y += nj.z * C.Dx[q];
                    B.z += nj.x * C.Dy[q] - nj.y * C.Dx[q];
                }
            }
        }
    }
    const T kn = C.K2 * (Q.Kax[0] * ni.x + Q.Kax[1] * ni.y + Q.Kax[2] * ni.z);
    B.x += kn * Q.Kax[0];
    B.y += kn * Q.Kax[1];
    B.z += kn * Q.Kax[2];
#pragma unroll
    for (int s = 0; s < SH::NS; ++s) {
        B.x += C.J[s] * acc[s].x;
        B.y += C.J[s] * acc[s].y;
        B.z += C.J[s] * acc[s].z;
    }
    return B;
}

// The field of one site from its neighbours' cells, cell(q) giving bond q's.
template <typename T, int S, int NDMI, typename Cell>
__device__ __forceinline__ V3<T> shape_B_of(const StepCoef<T>& C, const Site2D<T>& Q, Cell cell, V3<T> ni,
                                            V3<T> base) {
    using SH = ShapeTab<S>;
    V3<T> acc[SH::NS];
    V3<T> B = base;
#pragma unroll
    for (int q = 0; q < SH::NB; ++q) {
        const V3<T> nj = cell(q);
        const int sh = SH::sh[q];
        if (first_of_shell<SH>(q)) acc[sh] = nj;
        else acc[sh] = acc[sh] + nj;
        if (q < NDMI) {
            // + n_j x D with D = (Dx, Dy, 0)
            B.x -= nj.z * C.Dy[q];
            B.y += nj.z * C.Dx[q];
            B.z += nj.x * C.Dy[q] - nj.y * C.Dx[q];
        }
    }
    const T kn = C.K2 * (Q.Kax[0] * ni.x + Q.Kax[1] * ni.y + Q.Kax[2] * ni.z);
    B.x += kn * Q.Kax[0];
    B.y += kn * Q.Kax[1];
    B.z += kn * Q.Kax[2];
#pragma unroll
    for (int s = 0; s < SH::NS; ++s) {
        B.x += C.J[s] * acc[s].x;
        B.y += C.J[s] * acc[s].y;
        B.z += C.J[s] * acc[s].z;
    }
    return B;
}

// shape_B_of with the neighbours' cells by index (nb[q]).
template <typename T, int S, int NDMI>
__device__ __forceinline__ V3<T> shape_B_cells(const StepCoef<T>& C, const Site2D<T>& Q, const V4<T>* sv,
                                               const int (&nb)[ShapeTab<S>::NB], V3<T> ni, V3<T> base) {
    return shape_B_of<T, S, NDMI>(C, Q, [&](int q) { return lds_cell_xyz(sv, nb[q]); }, ni, base);
}

struct TileMap {
    int tiles_x, tiles_y;
    int xcd_bands;   // 1: XCD-banded mapping (tile count divisible by 8), 0: identity
};

// Element at a 32-bit byte offset from a base: the address is the base plus
// the zero-extended offset, which the compiler issues as a scalar-base
// load or store with a 32-bit vector offset.
template <typename T>
__device__ __forceinline__ T at_byte(const T* base, uint32_t off) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + off);
}
template <typename T>
__device__ __forceinline__ T* ptr_byte(T* base, uint32_t off) {
    return reinterpret_cast<T*>(reinterpret_cast<char*>(base) + off);
}

// Periodic wrap (or open-boundary rejection) of a staged coordinate.  A tile
// plus halo can be more than twice as wide as a small lattice, so the wrap
// is a full modulo, not a single +-n.
__device__ __forceinline__ int wrap_once(int g, int n, int per, bool& in) {
    if (g >= 0 && g < n) return g;
    if (!per) {
        in = false;
        return 0;
    }
    g %= n;
    return g < 0 ? g + n : g;
}

template <typename T, int S, int TX, int TY>
struct TileLDS {
    static constexpr int R = ShapeTab<S>::R;
    static constexpr int WN = TX + 4 * R, HN = TY + 4 * R;
    static constexpr int WP = TX + 2 * R, HP = TY + 2 * R;
    static constexpr int PN = WN * HN, PP = WP * HP, PT = TX * TY;
    V4<T> sN[PN];
    V4<T> sP[PP];
};

// Boundary form of a tile instance (PER): 0 any boundary; 1 both axes
// periodic; 2 both axes periodic with power-of-two sides, where the wrap is
// one mask (in the general form every wave with a cell past an edge runs a
// remainder of some 25 instructions, three to five times per step).
template <int PER>
__device__ __forceinline__ int wrap_cell(int g, int n, int per, bool& in) {
    if constexpr (PER == 2) return g & (n - 1);
    else return wrap_once(g, n, PER ? 1 : per, in);
}
// Site of cell (gx, gy) of a lattice na wide.
template <int PER>
__device__ __forceinline__ int cell_index(int gx, int gy, int na) {
    if constexpr (PER == 2) return gx + (gy << (31 - __builtin_clz(na)));
    else return gx + gy * na;
}

// Global site of the predictor-frame cell (px, py), or in = false for a
// cell outside an open lattice (PER: both axes periodic, never).
template <typename T, int S, int TX, int TY, int PER = 0>
__device__ __forceinline__ int cell_site(const Site2D<T>& Q, int x0, int y0, int px, int py, bool& in) {
    constexpr int R = ShapeTab<S>::R;
    in = true;
    const int gx = wrap_cell<PER>(x0 - R + px, Q.na, Q.per_a, in);
    const int gy = wrap_cell<PER>(y0 - R + py, Q.nb, Q.per_b, in);
    return cell_index<PER>(gx, gy, Q.na);
}

// External plus thermal field of a predictor-frame cell (the base of
// shape_B_aos): depends only on the site, the step and the seed, so it is
// formed while the spins are still in flight.  The empty asm keeps the draw
// behind its branch: where nothing else in it needs one (periodic sides that
// are powers of two) the compiler drew the field for every step and selected
// afterwards, which made steps at T = 0 cost what those at T > 0 do (256 x 256,
// three triangular shells with DMI: 5.07 us, now 4.58; at T > 0 5.24 and 5.14).
template <typename T, int S, int TX, int TY, int PER = 0>
__device__ __forceinline__ V3<T> cell_base(const StepCoef<T>& C, const Site2D<T>& Q, const LLGArgs<T>& A, int x0,
                                           int y0, int px, int py) {
    bool in;
    const int site = cell_site<T, S, TX, TY, PER>(Q, x0, y0, px, py, in);
    const V3<T> Bext{C.Bext[0], C.Bext[1], C.Bext[2]};
    if (!A.thermal || !in) return Bext;
    asm volatile("");
    return Bext + Q.sigma * normals3(thermal_bits(A.key, (uint32_t)site), T(0));
}

// Ring cell h (0 <= h < ring size) of the predictor frame: R rows above and
// below the tile, then R columns left and right of each tile row.
template <int R, int TX, int TY>
__device__ __forceinline__ void ring_cell(int h, int& px, int& py) {
    constexpr int WP = TX + 2 * R;
    if (h < 2 * R * WP) {
        const int r = h / WP;
        px = h - r * WP;
        py = r < R ? r : TY + r;
    } else {
        const int k = h - 2 * R * WP;
        const int r = k / (2 * R), q = k - r * (2 * R);
        py = R + r;
        px = q < R ? q : TX + q;
    }
}

// Predictor of one predictor-frame cell (px, py) with its external plus
// thermal field base.  Writes to sP what the corrector's field is evaluated on and returns
// what the corrector needs of the site itself:
//   Depondt: n^p = R(A) n, returns w = B + alpha n x B (A = -gp w);
//   Heun:    n^p = (n + dt n x A) / |...|, returns f = n x A;
//   SIB:     x solves the midpoint stage with A frozen; sP holds the
//            midpoint m = (n + x)/2 (Appendix C), returns nothing.
// Cells that fall outside an open lattice hold a zero spin.
template <typename T, int S, int NDMI, int TX, int TY, int SOLVER, int PER = 0>
__device__ __forceinline__ V3<T> predict_cell(const StepCoef<T>& C, const Site2D<T>& Q, const LLGArgs<T>& A, int x0,
                                              int y0, int px, int py, TileLDS<T, S, TX, TY>& L, V3<T> base) {
    using TL = TileLDS<T, S, TX, TY>;
    constexpr int R = TL::R, WN = TL::WN, WP = TL::WP;
    bool in;
    cell_site<T, S, TX, TY, PER>(Q, x0, y0, px, py, in);
    V4<T> out{T(0), T(0), T(0), T(0)};
    V3<T> keep{T(0), T(0), T(0)};
    if (in) {
        const int c = (py + R) * WN + (px + R);
        const V3<T> ni = lds_cell_xyz(L.sN, c);
        const V3<T> B = shape_B_aos<T, S, NDMI, WN>(C, Q, L.sN, c, ni, base);
        V3<T> o;
        if constexpr (SOLVER == SOLVER_HEUN) {
            keep = cross(ni, llg_A(ni, B, A.gp, A.alpha));
            o = normalize3(ni + A.dt * keep);
        } else if constexpr (SOLVER == SOLVER_SIB) {
            o = T(0.5) * (ni + sib_stage(ni, llg_A(ni, B, A.gp, A.alpha), A.dt));
        } else {
            keep = llg_w(ni, B, A.alpha);
            // n^p only feeds the corrector's field; its FP32 length error
            // (~1 ulp) is left in place, only n(t+dt) is renormalised.
            o = rotate_half(ni, keep, rot_half_factor(A.gp, A.dt));
        }
        out = V4<T>{o.x, o.y, o.z, T(0)};
    }
    L.sP[py * WP + px] = out;
    return keep;
}

// Corrector of tile site (tx, ty) from the predictor cells in sP, the spin
// n(t) in sN and what the predictor kept for the site (w or n x A, and the
// external plus thermal field): returns n(t+dt).
template <typename T, int S, int NDMI, int TX, int TY, int SOLVER>
__device__ __forceinline__ V3<T> correct_cell(const StepCoef<T>& C, const Site2D<T>& Q, const LLGArgs<T>& A, int tx,
                                              int ty, const TileLDS<T, S, TX, TY>& L, V3<T> keepA, V3<T> keepB) {
    using TL = TileLDS<T, S, TX, TY>;
    constexpr int R = TL::R, WN = TL::WN, WP = TL::WP;
    const int c = (ty + R) * WP + (tx + R);
    const V3<T> npi = lds_cell_xyz(L.sP, c);
    const V3<T> B = shape_B_aos<T, S, NDMI, WP>(C, Q, L.sP, c, npi, keepB);
    const V3<T> ni = lds_cell_xyz(L.sN, (ty + 2 * R) * WN + (tx + 2 * R));
    if constexpr (SOLVER == SOLVER_HEUN) {
        // n + dt (f(n) + f(n^p)) / 2, renormalised
        return normalize3(ni + (T(0.5) * A.dt) * (keepA + cross(npi, llg_A(npi, B, A.gp, A.alpha))));
    } else if constexpr (SOLVER == SOLVER_SIB) {
        // npi is the midpoint m; A(m) drives the second midpoint stage
        return renorm_if_float(sib_stage(ni, llg_A(npi, B, A.gp, A.alpha), A.dt));
    } else {
        // about the mean of the two rotation vectors (A + A^p)/2, up to -gp:
        // the sum turned by half the angle factor (the halving is exact)
        const V3<T> wp = llg_w(npi, B, A.alpha);
        return renorm_if_float(rotate_half(ni, keepA + wp, T(0.5) * rot_half_factor(A.gp, A.dt)));
    }
}

// One Depondt step of the TX x TY tile at (x0, y0) of one lattice.  Thread
// t owns tile sites t + j NT: it computes their predictor, keeps A and the
// thermal field in registers, and computes their corrector; the ring of
// predictor cells around the tile is shared out over the threads between.
template <typename T, int S, int NDMI, int TX, int TY, int NT, int SOLVER = SOLVER_DEPONDT, int PER = 0>
__device__ __forceinline__ void fused2d_tile(const StepCoef<T>& C, const Site2D<T>& Q, const LLGArgs<T>& A,
                                             int x0, int y0, const T* __restrict__ n, T* __restrict__ nout,
                                             TileLDS<T, S, TX, TY>& L) {
    using TL = TileLDS<T, S, TX, TY>;
    constexpr int R = TL::R, WN = TL::WN, WP = TL::WP, PN = TL::PN, PP = TL::PP, PT = TL::PT;
    static_assert(PT % NT == 0, "tile sites must divide evenly over the threads");
    constexpr int KPT = PT / NT;
    constexpr int RING = PP - PT;
    constexpr int KST = (PN + NT - 1) / NT;     // staged cells per thread
    constexpr int KRG = (RING + NT - 1) / NT;   // ring cells per thread
    const int N = Q.na * Q.nb;
    const int tid = threadIdx.x;

    // 1) load n(t) on the tile plus 2R halo into registers
    V3<T> st[KST];
#pragma unroll
    for (int k = 0; k < KST; ++k) {
        const int idx = tid + k * NT;
        // (cells past the staged frame are never stored)
        if constexpr (PER == 0) st[k] = V3<T>{T(0), T(0), T(0)};
        if (idx < PN) {
            const int ly = idx / WN, lx = idx - ly * WN;
            bool in = true;
            const int gx = wrap_cell<PER>(x0 - 2 * R + lx, Q.na, Q.per_a, in);
            const int gy = wrap_cell<PER>(y0 - 2 * R + ly, Q.nb, Q.per_b, in);
            if (in) {
                const int g = cell_index<PER>(gx, gy, Q.na);
                if constexpr (PER != 0) {
                    // 32-bit byte offsets (the host takes this instance only
                    // when 3N values have them)
                    const uint32_t b = (uint32_t)g * (uint32_t)sizeof(T);
                    st[k] = V3<T>{at_byte(n, b), at_byte(n + N, b), at_byte(n + 2 * N, b)};
                } else {
                    st[k] = V3<T>{n[g], n[N + g], n[2 * N + g]};
                }
            }
        }
    }
    // 2) external plus thermal fields of the owned cells while the loads are in flight
    V3<T> keepB[KPT], ringB[KRG];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int t = tid + j * NT;
        const int ty = t / TX, tx = t - ty * TX;
        keepB[j] = cell_base<T, S, TX, TY, PER>(C, Q, A, x0, y0, tx + R, ty + R);
    }
#pragma unroll
    for (int k = 0; k < KRG; ++k) {
        const int h = tid + k * NT;
        ringB[k] = V3<T>{T(0), T(0), T(0)};
        if (h < RING) {
            int px, py;
            ring_cell<R, TX, TY>(h, px, py);
            ringB[k] = cell_base<T, S, TX, TY, PER>(C, Q, A, x0, y0, px, py);
        }
    }
#pragma unroll
    for (int k = 0; k < KST; ++k) {
        const int idx = tid + k * NT;
        if (idx < PN) L.sN[idx] = V4<T>{st[k].x, st[k].y, st[k].z, T(0)};
    }
    __syncthreads();

    // 3) predictor: owned tile sites, then the ring of width R around the tile
    V3<T> keepA[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int t = tid + j * NT;
        const int ty = t / TX, tx = t - ty * TX;
        keepA[j] = predict_cell<T, S, NDMI, TX, TY, SOLVER, PER>(C, Q, A, x0, y0, tx + R, ty + R, L, keepB[j]);
    }
#pragma unroll
    for (int k = 0; k < KRG; ++k) {
        const int h = tid + k * NT;
        if (h < RING) {
            int px, py;
            ring_cell<R, TX, TY>(h, px, py);
            predict_cell<T, S, NDMI, TX, TY, SOLVER, PER>(C, Q, A, x0, y0, px, py, L, ringB[k]);
        }
    }
    __syncthreads();

    // 4) corrector on the owned tile sites
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        const int t = tid + j * NT;
        const int ty = t / TX, tx = t - ty * TX;
        const int gx = x0 + tx, gy = y0 + ty;
        if (gx >= Q.na || gy >= Q.nb) continue;
        const V3<T> o = correct_cell<T, S, NDMI, TX, TY, SOLVER>(C, Q, A, tx, ty, L, keepA[j], keepB[j]);
        const int gi = cell_index<PER>(gx, gy, Q.na);
        if constexpr (PER != 0) {
            const uint32_t b = (uint32_t)gi * (uint32_t)sizeof(T);
            store_out(ptr_byte(nout, b), o.x);
            store_out(ptr_byte(nout + N, b), o.y);
            store_out(ptr_byte(nout + 2 * N, b), o.z);
        } else {
            store_out(nout + gi, o.x);
            store_out(nout + N + gi, o.y);
            store_out(nout + 2 * N + gi, o.z);
        }
    }
}

// PER != 0: both axes periodic, so the boundary tests and zero fills of cells
// outside the lattice are compiled out, and spins are addressed by 32-bit
// byte offsets (the host takes it only when 3N values have them).
template <typename T, int S, int NDMI, int TX, int TY, int NT, int SOLVER = SOLVER_DEPONDT, int PER = 0>
__global__ void __launch_bounds__(NT) k_fused2d_shape(StepCoef<T> C, Site2D<T> Q, LLGArgs<T> A_arg, TileMap M,
                                                      const int* __restrict__ abort_flag, const T* __restrict__ n,
                                                      T* __restrict__ nout) {
    if (abort_flag && *abort_flag) return;
    const LLGArgs<T> A = resolve_step(A_arg);
    __shared__ TileLDS<T, S, TX, TY> L;
    const int ntiles = M.tiles_x * M.tiles_y;
    int tile = blockIdx.x;
    if (M.xcd_bands) tile = (blockIdx.x & 7) * (ntiles >> 3) + (blockIdx.x >> 3);
    const int ty0 = tile / M.tiles_x;
    fused2d_tile<T, S, NDMI, TX, TY, NT, SOLVER, PER>(C, Q, A, (tile - ty0 * M.tiles_x) * TX, ty0 * TY, n, nout, L);
}

// ------------------------------------------------------------ replica batch
// Many independent replicas that share one Hamiltonian (same stencil and
// coefficients) but differ in size, temperature, damping, time step and
// Philox replica index.
template <typename T>
struct ReplicaDesc {
    T* n[2];          // spin buffers (double-buffered for tiled replicas)
    int na, nb, per_a, per_b;
    int tiles_x;      // tiled replicas: tiles along a
    int thermal;
    T sigma, gp, alpha, dt;
    uint32_t seed_lo, seed_hi, replica;
};

template <typename T>
__device__ __forceinline__ void replica_args(const ReplicaDesc<T>& R, unsigned long long step, Site2D<T>& Q,
                                             LLGArgs<T>& A) {
    Q.na = R.na;
    Q.nb = R.nb;
    Q.per_a = R.per_a;
    Q.per_b = R.per_b;
    Q.sigma = R.sigma;
    A.gp = R.gp;
    A.alpha = R.alpha;
    A.dt = R.dt;
    A.thermal = R.thermal;
    A.key.seed_lo = R.seed_lo;
    A.key.seed_hi = R.seed_hi;
    A.key.step_lo = (uint32_t)step;
    A.key.step_hi = (uint32_t)(step >> 32);
    A.key.replica = R.replica;
}

// A tile of a tiled replica, with the replica's own description (one load
// between the kernel arguments and the spins).
template <typename T>
struct BatchWork {
    ReplicaDesc<T> r;
    int x0, y0;
    int form;            // boundary form (PER)
};

constexpr int kMixedForms = 3;   // PER of a batch whose tiles have different forms

// One Depondt step of every tile of every tiled replica: work item
// (replica, tile) per workgroup, in the form PER or, with kMixedForms, each in
// its own.  The step number is *step_base + k, so a
// captured graph of k = 0..K-1 can be replayed after step_base advances.
template <typename T, int S, int NDMI, int TX, int TY, int NT, int PER>
__global__ void __launch_bounds__(NT) k_batch_tiled(StepCoef<T> C, Site2D<T> Q, const BatchWork<T>* __restrict__ work,
                                                    const unsigned long long* __restrict__ step_base, int k,
                                                    int parity) {
    __shared__ TileLDS<T, S, TX, TY> L;
    const BatchWork<T> W = work[blockIdx.x];
    LLGArgs<T> A;
    replica_args(W.r, *step_base + (unsigned long long)k, Q, A);
    const bool odd = (parity ^ (k & 1)) != 0;
    T* const b0 = W.r.n[0];
    T* const b1 = W.r.n[1];
    const T* const in = odd ? b1 : b0;
    T* const out = odd ? b0 : b1;
    if constexpr (PER == kMixedForms) {
        switch (W.form) {
            case 0: fused2d_tile<T, S, NDMI, TX, TY, NT, SOLVER_DEPONDT, 0>(C, Q, A, W.x0, W.y0, in, out, L); break;
            case 1: fused2d_tile<T, S, NDMI, TX, TY, NT, SOLVER_DEPONDT, 1>(C, Q, A, W.x0, W.y0, in, out, L); break;
            default: fused2d_tile<T, S, NDMI, TX, TY, NT, SOLVER_DEPONDT, 2>(C, Q, A, W.x0, W.y0, in, out, L);
        }
    } else {
        fused2d_tile<T, S, NDMI, TX, TY, NT, SOLVER_DEPONDT, PER>(C, Q, A, W.x0, W.y0, in, out, L);
    }
}

// Resident replicas: one workgroup holds a whole LX x LY replica (sides powers
// of two) in LDS, as 16-byte cells, and advances it n_steps Depondt steps
// without touching HBM in between.  Each thread owns the sites tid + j*NT and
// keeps their spin, rotation vector w and thermal field in registers.  The
// cells lie in a frame of zero cells as wide as the stencil, which open edges
// read; neighbours past periodic edges are read from the other side, so a
// step has two barriers and no images to refresh.
//
// What bounds it is the instructions of one CU (and, with four sites a thread,
// the 128 registers of a 1024-thread workgroup), so a neighbour should cost no
// more than its read: the cell is one of 2R+1 columns, wrapped once per launch,
// plus a constant, as a thread's rows lie NT/LX apart and only those of the
// first and the last can leave the lattice; theirs add a row offset that is
// the same for a whole wavefront of LX = 64.  Wrapping each neighbour's index
// by masks, with tests for open edges, took 13.5 us a step for 64^2 with the
// 18 bonds of three triangular shells and DMI (81 registers spilled), this
// 7.3 us (18 bonds, 32^2: 2.03 and 1.92; four bonds: 3.80 and 3.90 for 64^2,
// 1.10 and 1.14 for 32^2).  The frame of 64^2 is two cells wide for a reach of
// one too: it leaves less of a CU's LDS than a tiled workgroup needs, which
// beside a resident one, whose chain of steps the batch waits for, cost 1190
// instead of 1020 us (128 steps, sides 32 to 256).
template <typename T, int S, int NDMI, int LX, int LY, int NT>
__global__ void __launch_bounds__(NT) k_batch_resident(StepCoef<T> C, Site2D<T> Q,
                                                       const ReplicaDesc<T>* __restrict__ reps,
                                                       const int* __restrict__ list,
                                                       const unsigned long long* __restrict__ step_base,
                                                       int n_steps) {
    using SH = ShapeTab<S>;
    constexpr int N = LX * LY, PT = N / NT, RP = NT / LX, R = SH::R, F = PT > 1 ? 2 : R, W = LX + 2 * F, P = W * (LY + 2 * F);
    static_assert(N % NT == 0 && NT % LX == 0, "whole sites per thread, whole rows between them");
    static_assert((LX & (LX - 1)) == 0 && (LY & (LY - 1)) == 0 && RP >= R, "sides wrap by a mask");
    static_assert(F >= R, "a frame as wide as the reach");
    __shared__ V4<T> sN[P];
    __shared__ V4<T> sP[P];
    const ReplicaDesc<T> Rp = reps[list[blockIdx.x]];
    LLGArgs<T> A;
    const unsigned long long first = *step_base;
    replica_args(Rp, first, Q, A);
    const int tid = threadIdx.x;
    T* g = Rp.n[0];
    for (int c = tid; c < P; c += NT) sN[c] = sP[c] = V4<T>{T(0), T(0), T(0), T(0)};
    __syncthreads();
    const int x = tid & (LX - 1);
    const int y0 = LX % 64 == 0 ? __builtin_amdgcn_readfirstlane(tid / LX) : tid / LX;
    const int c0 = (y0 + F) * W + F + x;
    V3<T> ni[PT], base[PT], keep[PT];
#pragma unroll
    for (int j = 0; j < PT; ++j) {
        ni[j] = load3(g, N, tid + j * NT);
        sN[c0 + j * RP * W] = V4<T>{ni[j].x, ni[j].y, ni[j].z, T(0)};
    }
    __syncthreads();
    int col[2 * R + 1];            // row y0, columns x-R..x+R
#pragma unroll
    for (int d = -R; d <= R; ++d) col[d + R] = c0 - x + (Q.per_a ? (x + d) & (LX - 1) : x + d);
    int below[R], above[R];        // rows past the first and the last one, seen from row y0
#pragma unroll
    for (int d = 1; d <= R; ++d) {
        const int lo = y0 - d, hi = y0 + (PT - 1) * RP + d;
        below[d - 1] = ((Q.per_b ? lo & (LY - 1) : lo) - y0) * W;
        above[d - 1] = ((Q.per_b ? hi & (LY - 1) : hi) - y0) * W;
    }
    auto cell = [&](const V4<T>* sv, int j, int q) {
        const int da = SH::da[q], db = SH::db[q];
        int row = (j * RP + db) * W;
        if (j == 0 && db < 0) row = below[-db - 1];
        if (j == PT - 1 && db > 0) row = above[db - 1];
        return lds_cell_xyz(sv, col[da + R] + row);
    };
    const V3<T> Bext{C.Bext[0], C.Bext[1], C.Bext[2]};
    const T h = rot_half_factor(A.gp, A.dt);
    for (int k = 0; k < n_steps; ++k) {
        // the sums of columns and rows are formed where they are used: all
        // of them, held over the steps, spilled 38 registers with 18 bonds
        if constexpr (LX % 64 == 0 && SH::NB > 4) {
#pragma unroll
            for (int d = 0; d < R; ++d) asm volatile("" : "+s"(below[d]), "+s"(above[d]));
        }
        A.key.step_lo = (uint32_t)(first + k);
        A.key.step_hi = (uint32_t)((first + k) >> 32);
        V3<T> p[PT];
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            base[j] = Bext;
            if (A.thermal) {
                asm volatile("");   // the draw stays behind the branch
                base[j] = base[j] + Q.sigma * normals3(thermal_bits(A.key, (uint32_t)(tid + j * NT)), T(0));
            }
            auto nb = [&](int q) { return cell(sN, j, q); };
            keep[j] = llg_w(ni[j], shape_B_of<T, S, NDMI>(C, Q, nb, ni[j], base[j]), A.alpha);
            p[j] = rotate_half(ni[j], keep[j], h);
            sP[c0 + j * RP * W] = V4<T>{p[j].x, p[j].y, p[j].z, T(0)};
            __builtin_amdgcn_sched_barrier(0);   // one site's cells in registers at a time
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            auto nb = [&](int q) { return cell(sP, j, q); };
            const V3<T> wp = llg_w(p[j], shape_B_of<T, S, NDMI>(C, Q, nb, p[j], base[j]), A.alpha);
            ni[j] = renorm_if_float(rotate_half(ni[j], keep[j] + wp, T(0.5) * h));
            sN[c0 + j * RP * W] = V4<T>{ni[j].x, ni[j].y, ni[j].z, T(0)};
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < PT; ++j) store3(g, N, tid + j * NT, ni[j]);
}

__global__ void k_advance_step(unsigned long long* step_base, int k) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *step_base += (unsigned long long)k;
}

}  // namespace sp
