// Device-side building blocks of the relativistic PIC step for gfx950.
//
// Everything here is templated on the working precision R (float, double)
// and on the number of spatial dimensions D, so that the hot loops are
// straight-line code.  Particles carry positions relative to their tile
// centre; tiles are staged in LDS with a halo, so that interpolation reads
// and deposit atomics never leave the work-group's LDS.
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pic {

// ---------------------------------------------------------------- tables

// One entry per tile of every box.
struct TileDesc {
    int32_t box;
    int32_t tc[3];      // tile coordinates inside the box
    int32_t nt[3];      // tiles per dimension of the box
    int32_t n[3];       // cells per dimension of the box
    int64_t cell0;      // offset of the box's first cell in the field planes
    int32_t tile0;      // global id of the box's tile (0,0,0)
    int32_t walls;      // bit 0: conducting wall on the tile's low-x face
                        // (x = 0), bit 1: on its high-x face (x = n0)
};

// Launch-wide constants of the particle and field kernels.
template <typename R>
struct Params {
    const TileDesc *tiles;
    int32_t ntiles;
    int32_t nspecies;
    int32_t T[3];
    int32_t pad0;
    R c;                      // Courant number
    R inv_c;                  // 1 / c
    const R *charge;          // [box][species]
    const R *qm;              // [box][species] App. C factor s
    R *E, *B, *J;             // [3][cells_total]
    int64_t cells_total;
    R *pos, *u, *xold;        // [D|3][cap_total]
    int64_t cap_total;
    const int64_t *seg_off;   // [tile][species]
    const int32_t *seg_cap;
    int32_t *seg_cnt;
    R *jblk;                  // [tile*species][3][JV]
    R *ob_pos, *ob_u;         // [tile*species][D|3][ob_cap]
    int32_t *ob_dir;          // [tile*species][ob_dir_stride]
    int32_t *ob_cnt;          // [tile*species]
    int64_t ob_cap;
    int64_t ob_dir_stride;    // slots per outbox direction list (ob_cap)
    R *tmp;                   // sort staging [(D+3)][cap_total]
    int32_t *err;             // latched error bits
    int32_t *nf_seg;          // [tile*species] particles flagged near a cell face
    R nf_band[3];             // near-face band per dimension: 2 ulp(T_d/2) in R
    uint32_t species_mask;    // species the launch works on (bit s = species s)
    int32_t *mig_counts;      // [tile*species][ncodes] migration counts, or null
    int32_t *queue;           // work counter of the persistent walker
    int32_t *order;           // (tile, species) segments in visiting order
    int32_t *ids;             // [cap_total] origin of each particle, or null
    int32_t *ob_ids;          // [tile*species][ob_cap] origin of each leaver
    int32_t *ob_boff;         // [tile*species][ncodes+1] outbox bucket starts by direction code
    int32_t *ob_idx;          // [tile*species][ob_cap] outbox slots in bucket order
    int32_t lds_planes;       // the push keeps E and B in LDS as planes of their own (tiles
                              // whose interleaved rows cost a work-group), see FieldLds
    int32_t dir_lds;          // leavers whose direction code the push keeps in LDS
    R *bnext;                 // [3][cells_total] B after both half updates (whole step), or null
};

enum : int32_t { ERR_CAPACITY = 1, ERR_CFL = 2, ERR_NONFINITE = 4, ERR_OUT_OF_TILE = 8, ERR_ADJ_MAP = 16 };

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ int wrapi(int i, int n)
{
    int r = i % n;
    return r < 0 ? r + n : r;
}

// The same for a reach below one box length, without the division.
__device__ __forceinline__ int wrap_once(int i, int n)
{
    return i < 0 ? i + n : (i >= n ? i - n : i);
}

// The same for a halo that may be longer than a short box.
__device__ __forceinline__ int wrap_near(int i, int n)
{
    while (i < 0) i += n;
    while (i >= n) i -= n;
    return i;
}

// A value that every lane of the wave holds, in scalar registers (a load after
// stores stays a vector load, even from one address).
template <typename V>
__device__ __forceinline__ V uniform(V v)
{
    int w[sizeof(V) / 4];
    __builtin_memcpy(w, &v, sizeof(V));
#pragma unroll
    for (int k = 0; k < (int)(sizeof(V) / 4); ++k) w[k] = __builtin_amdgcn_readfirstlane(w[k]);
    __builtin_memcpy(&v, w, sizeof(V));
    return v;
}

// Tile (or (tile, species) segment) of this work-group in launches with one
// work-group per tile (or segment), out of n.  The
// dispatcher hands consecutive work-groups to the eight dies (XCDs, each
// with its own L2) in turn; this bijection gives every die a contiguous
// range of tiles instead, so that neighbouring tiles, which share cache
// lines of the field planes and each other's halos, meet in one L2.
__device__ __forceinline__ int xcd_tile(int b, int n)
{
    constexpr int NXCD = 8;
    const int x = b % NXCD, l = b / NXCD, per = n / NXCD, rem = n % NXCD;
    return x < rem ? x * (per + 1) + l : rem * (per + 1) + (x - rem) * per + l;
}

// Product of two small non-negative integers (LDS block indices and strides,
// both far below 2^23): v_mul_i32_i24 issues at the full VALU rate, the
// 32-bit v_mul_lo_u32 at a quarter of it.
__device__ __forceinline__ int imul24(int a, int b) { return (int)__umul24((unsigned)a, (unsigned)b); }

// k / n for a cell index inside a tile (k and n far below 2^20), from
// inv = 1.0f / n: (k + 1/2) / n lies at least 1/(2n) from an integer, more
// than the rounding of the product, so the truncation is exact.
__device__ __forceinline__ int div_small(int k, float inv) { return (int)(((float)k + 0.5f) * inv); }

// Loads and stores at a 32-bit byte offset from a uniform base pointer: the
// memory instruction adds the 64-bit scalar base and the 32-bit vector
// offset itself, so a particle index costs one shift for every plane.
template <typename T>
__device__ __forceinline__ T ld_off(const T *base, uint32_t off)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + off);
}
template <typename T>
__device__ __forceinline__ void st_off(T *base, uint32_t off, T v)
{
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + off) = v;
}

template <int D>
__device__ __forceinline__ int ext(const int32_t T[3], int d, int halo)
{
    return d < D ? T[d] + halo : 1;
}

// Number of lanes below this one whose bit is set in mask.
__device__ __forceinline__ int lanes_below(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Near-face flag of a stored tile-local position: some grid coordinate lies
// within band_d of an integer (a cell face).  x - rint(x) is exact in R, so
// the test is the same in any precision that holds x exactly.
template <typename R, int D>
__device__ __forceinline__ bool near_face(const R x[3], const R band[3])
{
    bool f = false;
#pragma unroll
    for (int d = 0; d < D; ++d) f = f || fabs(x[d] - rint(x[d])) <= band[d];
    return f;
}

// The same flag as a sign: the smallest distance to a cell face less the
// band, <= 0 exactly when near_face holds (a difference of two floats has the
// sign of their comparison).
template <typename R, int D>
__device__ __forceinline__ R face_distance(const R x[3], const R band[3])
{
    R m = fabs(x[0] - rint(x[0])) - band[0];
#pragma unroll
    for (int d = 1; d < D; ++d) m = fmin(m, fabs(x[d] - rint(x[d])) - band[d]);
    return m;
}

__device__ __forceinline__ void latch(int32_t *err, int32_t bits)
{
    atomicOr(err, bits);
}

// OR the per-thread error bits of a wave into the device word with one
// atomic (called by every lane of the wave): a burst of failing particles
// then costs one atomic per wave instead of one per particle.
__device__ __forceinline__ void latch_wave(int32_t *err, int32_t bits)
{
    const unsigned long long any = __ballot(bits != 0);
    if (!any) return;
    int v = bits;
    for (int o = 32; o > 0; o >>= 1) v |= __shfl_xor(v, o);
    if ((int)(threadIdx.x & 63) == __ffsll((long long)any) - 1) atomicOr(err, v);
}

// LDS atomic add of a current value computed in precision R into an
// accumulator of type A.  A = float or double: a floating-point add.
// A = long long (FP32 runs): fixed point.  The deposit's charge is scaled by
// 2^e (fixed_exponent, |q| 2^e in [2^29, 2^30)) so that every ZigZag value
// has magnitude below 2^31; the value is truncated to an integer (an error
// below one unit, 2^-29 |q|, under the FP32 rounding of a value of a tenth
// of |q|) and added exactly, so a block does not depend on the order of its
// atomics, and the 64-bit integer add of the LDS runs much faster than its
// FP64 add on gfx950.
template <typename A, typename R>
__device__ __forceinline__ void lds_add(A *p, R v)
{
    if constexpr (std::is_same<A, long long>::value) {
        static_assert(sizeof(R) == 4, "fixed-point accumulation is for FP32 values");
        atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)(long long)(int)v);
    } else {
        atomicAdd(p, (A)v);
    }
}

// Exponent e of the fixed-point scale 2^e of one segment's current block:
// |q| 2^e < 2^30, so that ZigZag values (at most (1 + 1/12) |q| per
// segment) stay below 2^31; an entry then sums at most 4 segments per
// particle, so 2^30 particles fit in 64 bits.
template <typename R>
__device__ __forceinline__ int fixed_exponent(R q)
{
    return q == R(0) ? 0 : 29 - ilogb(q);
}

// Strides of a block of vector components in LDS, in elements: from one
// component to the next, along y and along z (along x: 1).
struct Strides {
    int m, y, z;
};

// Field halo block in LDS: local cells -1..T per grid dimension.
template <int D>
struct FieldBox {
    int e0, e1, e2;   // extents
    int n;            // cells in the block
    __device__ FieldBox(const int32_t T[3])
    {
        e0 = ext<D>(T, 0, 2);
        e1 = ext<D>(T, 1, 2);
        e2 = ext<D>(T, 2, 2);
        n = e0 * e1 * e2;
    }
    __device__ __forceinline__ Strides planes() const { return {n, e0, e0 * e1}; }
};

// Current halo block: local cells -1..T+1 per grid dimension.
template <int D>
struct CurBox {
    int e0, e1, e2;
    int n;
    __device__ CurBox(const int32_t T[3])
    {
        e0 = ext<D>(T, 0, 3);
        e1 = ext<D>(T, 1, 3);
        e2 = ext<D>(T, 2, 3);
        n = e0 * e1 * e2;
    }
    // Strides of a block over these cells whose rows along x hold NC
    // components one after another, [row][NC][e0]: component, y row, z layer.
    template <int NC>
    __device__ __forceinline__ Strides rows() const
    {
        return {e0, NC * e0, NC * e0 * e1};
    }
    // every component in a plane of its own, [3][n]
    __device__ __forceinline__ Strides planes() const { return {n, e0, e0 * e1}; }
    // the current block, in LDS and in memory
    __device__ __forceinline__ Strides current() const { return rows<3>(); }
};

// Where the push keeps E and B in LDS (elements of sF).  1D and 2D: rows of
// all six components, [row][6][e0].  The components and the next row of a cell
// then lie within the 255 elements that one LDS read pair reaches by its
// immediate offsets, so a particle's 12 (2D) read pairs share four base
// addresses (2D FP32 push: 331 VALU instructions per 64 particles against 371
// with one plane per component).  3D: one plane per component.  A z layer
// lies beyond those offsets in any case, and rows of 66 elements map an 8 x 8
// plane of cells, which an ordered plasma keeps in one wave, onto few banks (8^3
// tiles, FP32, walls: push 611 us with rows, 587 us with planes).  Planes
// also in 1D and 2D tiles where the larger rows would cost a CU a work-group.
template <int D>
struct FieldLds {
    Strides e, b;
    int b0;          // offset of Bx's block
    __device__ FieldLds(const CurBox<D> &cb, const FieldBox<D> &fb, bool planes)
    {
        e = b = cb.template rows<6>();
        b0 = 3 * cb.e0;
        if (planes) {
            e = cb.planes();
            b = fb.planes();
            b0 = 3 * cb.n;
        }
    }
};

// Cell coordinates of entry k of a block of extents e0, e1 (x fastest).
template <int D>
__device__ __forceinline__ void cell_of(int k, int e0, int e1, float inv0, float inv1, int &lx, int &ly, int &lz)
{
    const int r = D > 1 ? div_small(k, inv0) : 0;
    lz = D > 2 ? div_small(r, inv1) : 0;
    lx = D > 1 ? k - imul24(r, e0) : k;
    ly = D > 2 ? r - imul24(lz, e1) : r;
}

// Storage index of the cell at local coordinates lx-1.. of the tile; a halo
// reaches at most one box length beyond the box (every edge is >= 2).
template <int D>
__device__ __forceinline__ int64_t halo_cell(const TileDesc &td, const int32_t T[3], int lx, int ly, int lz)
{
    int g[3] = {0, 0, 0};
    const int l[3] = {lx, ly, lz};
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int v = td.tc[d] * T[d] + l[d] - 1;
        g[d] = v < 0 ? v + td.n[d] : (v >= td.n[d] ? v - td.n[d] : v);
    }
    return td.cell0 + g[0] + (D > 1 ? (int64_t)td.n[0] * (D > 2 ? g[1] + (int64_t)td.n[1] * g[2] : g[1]) : 0);
}

// Copy three planes of the tile's halo block into LDS, periodic wrap; dst
// layout [3][bx.n].  NEG: with the opposite sign.
template <typename R, int D, bool NEG = false, typename BoxT>
__device__ __forceinline__ void stage_block(const R *__restrict__ src, int64_t N, const TileDesc &td,
                                            const int32_t T[3], R *dst, const BoxT &bx)
{
    const float inv0 = 1.0f / bx.e0, inv1 = 1.0f / bx.e1;
    for (int k = threadIdx.x; k < bx.n; k += blockDim.x) {
        int lx, ly, lz;
        cell_of<D>(k, bx.e0, bx.e1, inv0, inv1, lx, ly, lz);
        const int64_t g = halo_cell<D>(td, T, lx, ly, lz);
#pragma unroll
        for (int m = 0; m < 3; ++m) dst[m * bx.n + k] = NEG ? -src[m * N + g] : src[m * N + g];
    }
}

// E (local cells -1..T+1) and B (local cells -1..T) of the tile into the LDS
// block sF.  Two cells per thread and trip, all of their loads before the
// first LDS write: the staging is one or two memory latencies.
template <typename R, int D>
__device__ __forceinline__ void stage_fields(const R *__restrict__ E, const R *__restrict__ B, int64_t N,
                                             const TileDesc &td, const int32_t T[3], R *sF, const CurBox<D> &cb,
                                             const FieldLds<D> &fl)
{
    constexpr int U = 2;
    const float inv0 = 1.0f / cb.e0, inv1 = 1.0f / cb.e1;
    for (int k0 = threadIdx.x; k0 < cb.n; k0 += U * blockDim.x) {
        R v[U][6];
        int at[U], bt[U];
        bool inb[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int k = k0 + j * blockDim.x;
            int lx, ly, lz;
            cell_of<D>(k, cb.e0, cb.e1, inv0, inv1, lx, ly, lz);
            at[j] = lx + imul24(ly, fl.e.y) + imul24(lz, fl.e.z);
            bt[j] = lx + imul24(ly, fl.b.y) + imul24(lz, fl.b.z) + fl.b0;
            inb[j] = k < cb.n && lx < T[0] + 2 && (D < 2 || ly < T[1] + 2) && (D < 3 || lz < T[2] + 2);
            if (k < cb.n) {
                const int64_t g = halo_cell<D>(td, T, lx, ly, lz);
#pragma unroll
                for (int m = 0; m < 3; ++m) v[j][m] = E[m * N + g];
                if (inb[j]) {
#pragma unroll
                    for (int m = 0; m < 3; ++m) v[j][3 + m] = B[m * N + g];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (k0 + j * (int)blockDim.x < cb.n) {
#pragma unroll
                for (int m = 0; m < 3; ++m) sF[at[j] + m * fl.e.m] = v[j][m];
                if (inb[j]) {
#pragma unroll
                    for (int m = 0; m < 3; ++m) sF[bt[j] + m * fl.b.m] = v[j][3 + m];
                }
            }
        }
    }
}

// First half of the B advance (push_half_b1) applied to the LDS copy of B:
// B -= h curl+ E on local cells -1..T, from the staged E (cells -1..T+1).
// With bnext, the tile's own cells also get their second half (push_half_b2,
// the same E) and go to the planes bnext: the stored B must stay as it is
// until every work-group has staged its halo, and the E update, which needs
// B after both halves, runs in the next launch.
template <typename R, int D>
__device__ __forceinline__ void half_b_lds(R *sB, const Strides sb, const FieldBox<D> &fb, const R *sE,
                                           const Strides se, R h, const TileDesc &td, const int32_t T[3], R *bnext,
                                           int64_t N)
{
    const float inv0 = 1.0f / fb.e0, inv1 = 1.0f / fb.e1;
    for (int k = threadIdx.x; k < fb.n; k += blockDim.x) {
        int lx, ly, lz;
        cell_of<D>(k, fb.e0, fb.e1, inv0, inv1, lx, ly, lz);
        const int e = lx + imul24(ly, se.y) + imul24(lz, se.z), f = lx + imul24(ly, sb.y) + imul24(lz, sb.z);
        const int ip = D > 0 ? 1 : 0, jp = D > 1 ? se.y : 0, kp = D > 2 ? se.z : 0;
        const R *Ex = sE, *Ey = sE + se.m, *Ez = sE + 2 * se.m;
        const R ex = Ex[e], ey = Ey[e], ez = Ez[e];
        const R cx = (Ez[e + jp] - ez) - (Ey[e + kp] - ey);
        const R cy = (Ex[e + kp] - ex) - (Ez[e + ip] - ez);
        const R cz = (Ey[e + ip] - ey) - (Ex[e + jp] - ex);
        const R bx = fma(-h, cx, sB[f]), by = fma(-h, cy, sB[f + sb.m]), bz = fma(-h, cz, sB[f + 2 * sb.m]);
        sB[f] = bx;
        sB[f + sb.m] = by;
        sB[f + 2 * sb.m] = bz;
        if (bnext) {
            const int ox = lx - 1, oy = D > 1 ? ly - 1 : 0, oz = D > 2 ? lz - 1 : 0;
            if (ox >= 0 && ox < T[0] && (D < 2 || (oy >= 0 && oy < T[1])) && (D < 3 || (oz >= 0 && oz < T[2]))) {
                const int64_t g = halo_cell<D>(td, T, lx, ly, lz);
                bnext[g] = fma(-h, cx, bx);
                bnext[N + g] = fma(-h, cy, by);
                bnext[2 * N + g] = fma(-h, cz, bz);
            }
        }
    }
}

// ---------------------------------------------------------- interpolation

// Per-particle interpolation state: for each grid dimension the LDS base
// index and weight of a node-centred (offset 0) and a half-cell (offset
// 1/2) sub-lattice.
template <typename R, int D>
struct Stencil {
    int bn[3], bh[3];
    R wn[3], wh[3];
};

template <typename R, int D>
__device__ __forceinline__ void make_stencil(const R x[3], const int32_t T[3], Stencil<R, D> &s)
{
#pragma unroll
    for (int d = 0; d < D; ++d) {
        R fl = floor(x[d]);
        int ci = (int)fl + T[d] / 2;      // cell in 0..T-1
        R f = x[d] - fl;
        s.bn[d] = ci + 1;                  // LDS offset of local cell -1 is 0
        s.wn[d] = f;
        bool up = f >= R(0.5);
        s.bh[d] = up ? ci + 1 : ci;
        s.wh[d] = up ? f - R(0.5) : f + R(0.5);
    }
}

// Linear interpolation at the LDS base b of one component (Ex..Bz, each from
// its own staggered sub-lattice: per dimension the half-cell lattice is used
// where the component is staggered by 1/2; weights w0, w1, w2 of the upper
// corners).
template <typename R, int D>
__device__ __forceinline__ R interp_at(const R *F, int b, const Strides st, R w0, R w1, R w2)
{
    const R *f = F + b;
    if constexpr (D == 1) {
        return f[0] * (R(1) - w0) + f[1] * w0;
    } else if constexpr (D == 2) {
        const R a0 = f[0] * (R(1) - w0) + f[1] * w0;
        const R a1 = f[st.y] * (R(1) - w0) + f[st.y + 1] * w0;
        return a0 * (R(1) - w1) + a1 * w1;
    } else {
        const R *g = f + st.z;
        const R a00 = f[0] * (R(1) - w0) + f[1] * w0;
        const R a10 = f[st.y] * (R(1) - w0) + f[st.y + 1] * w0;
        const R a01 = g[0] * (R(1) - w0) + g[1] * w0;
        const R a11 = g[st.y] * (R(1) - w0) + g[st.y + 1] * w0;
        const R c0 = a00 * (R(1) - w1) + a10 * w1;
        const R c1 = a01 * (R(1) - w1) + a11 * w1;
        return c0 * (R(1) - w2) + c1 * w2;
    }
}

// E and B at a particle from the block stage_fields filled.  Per dimension
// one node-centred and one half-cell base; a component's base is their sum.
template <typename R, int D>
__device__ __forceinline__ void interp_all(const R *sF, const FieldLds<D> &fl, const R x[3], const int32_t T[3],
                                           R e[3], R b[3])
{
    int n[3] = {0, 0, 0}, h[3] = {0, 0, 0}, bn[3] = {0, 0, 0}, bh[3] = {0, 0, 0};
    R wn[3] = {0, 0, 0}, wh[3] = {0, 0, 0};
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int s = d == 0 ? 1 : (d == 1 ? fl.e.y : fl.e.z), sb = d == 0 ? 1 : (d == 1 ? fl.b.y : fl.b.z);
        const R f0 = floor(x[d]);
        const int ci = (int)f0 + T[d] / 2 + 1;   // node-centred base: LDS offset of local cell -1 is 0
        const R f = x[d] - f0;
        const bool up = f >= R(0.5);
        n[d] = d == 0 ? ci : imul24(ci, s);
        h[d] = n[d] - (up ? 0 : s);
        bn[d] = d == 0 ? ci : imul24(ci, sb);
        bh[d] = bn[d] - (up ? 0 : sb);
        wn[d] = f;
        wh[d] = up ? f - R(0.5) : f + R(0.5);
    }
    const R *sB = sF + fl.b0;
    e[0] = interp_at<R, D>(sF, h[0] + n[1] + n[2], fl.e, wh[0], wn[1], wn[2]);
    e[1] = interp_at<R, D>(sF + fl.e.m, n[0] + h[1] + n[2], fl.e, wn[0], wh[1], wn[2]);
    e[2] = interp_at<R, D>(sF + 2 * fl.e.m, n[0] + n[1] + h[2], fl.e, wn[0], wn[1], wh[2]);
    b[0] = interp_at<R, D>(sB, bn[0] + bh[1] + bh[2], fl.b, wn[0], wh[1], wh[2]);
    b[1] = interp_at<R, D>(sB + fl.b.m, bh[0] + bn[1] + bh[2], fl.b, wh[0], wn[1], wh[2]);
    b[2] = interp_at<R, D>(sB + 2 * fl.b.m, bh[0] + bh[1] + bn[2], fl.b, wh[0], wh[1], wn[2]);
}

// ------------------------------------------------------------------ Boris

// Reciprocal and reciprocal square root in the working precision.  FP32
// uses the hardware v_rcp_f32 / v_rsq_f32 (about 1 ulp), which the FP32
// tolerance of the method admits; FP64 keeps correctly rounded division and
// square root.
template <typename R>
__device__ __forceinline__ R rcp_w(R x);
template <>
__device__ __forceinline__ float rcp_w<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <>
__device__ __forceinline__ double rcp_w<double>(double x) { return 1.0 / x; }
template <typename R>
__device__ __forceinline__ R rsqrt_w(R x);
template <>
__device__ __forceinline__ float rsqrt_w<float>(float x) { return __builtin_amdgcn_rsqf(x); }
template <>
__device__ __forceinline__ double rsqrt_w<double>(double x) { return 1.0 / sqrt(x); }

// Relativistic Boris update (App. C) of u^{n-1/2} -> u^{n+1/2}; velocities
// inside the update are carried in units of the Courant number c
// (inv_c = 1/c): u1 = c u + s E/2, gamma1 = sqrt(1 + |u1|^2/c^2),
// t = s B/(2 c gamma1), f = 2/(1+|t|^2), u2 = f (u1 + u1 x t),
// u3 = u1 + u2 x t + s E/2, u = u3/c.
// The multiply-adds are written out: the push and the adjoint's recomputation
// of it must round alike, or a particle within rounding of a face takes
// another branch of the deposit in one of them.
template <typename R>
__device__ __forceinline__ void boris(R u[3], const R e[3], const R b[3], R c, R inv_c, R s)
{
    const R hs = R(0.5) * s;
    auto norm2 = [](R x, R y, R z) -> R { return fma(z, z, fma(x, x, y * y)); };
    auto cross = [](R a, R d, R g, R h) -> R { return fma(a, d, -(g * h)); };   // a d - g h
    const R u1x = fma(c, u[0], hs * e[0]), u1y = fma(c, u[1], hs * e[1]), u1z = fma(c, u[2], hs * e[2]);
    const R k = (hs * inv_c) * rsqrt_w<R>(fma(inv_c * inv_c, norm2(u1x, u1y, u1z), R(1)));
    const R tx = k * b[0], ty = k * b[1], tz = k * b[2];
    const R f = R(2) * rcp_w<R>(R(1) + norm2(tx, ty, tz));
    const R u2x = f * (u1x + cross(u1y, tz, u1z, ty));
    const R u2y = f * (u1y + cross(u1z, tx, u1x, tz));
    const R u2z = f * (u1z + cross(u1x, ty, u1y, tx));
    u[0] = fma(hs, e[0], u1x + cross(u2y, tz, u2z, ty)) * inv_c;
    u[1] = fma(hs, e[1], u1y + cross(u2z, tx, u2x, tz)) * inv_c;
    u[2] = fma(hs, e[2], u1z + cross(u2x, ty, u2y, tx)) * inv_c;
}

// Lorentz factor of the implicit magnetic rotation: the gamma that solves
// w1 = w' + (w1/gamma) x tau, from gamma'^2 = 1 + |w'|^2/c^2 and
// u* = w'.tau/c (Vay 2008; Higuera and Cary 2017).  IEEE square roots in both
// precisions.
template <typename R>
__device__ __forceinline__ R implicit_gamma(const R w[3], const R tau[3], R inv_c)
{
    const R g2 = R(1) + (w[0] * w[0] + w[1] * w[1] + w[2] * w[2]) * (inv_c * inv_c);
    const R us = (w[0] * tau[0] + w[1] * tau[1] + w[2] * tau[2]) * inv_c;
    const R t2 = tau[0] * tau[0] + tau[1] * tau[1] + tau[2] * tau[2];
    const R sg = g2 - t2;
    return sqrt(R(0.5) * (sg + sqrt(sg * sg + R(4) * (t2 + us * us))));
}

// w <- (w + (w.t) t + w x t) / (1 + |t|^2): the exact rotation of the
// implicit update.
template <typename R>
__device__ __forceinline__ void exact_rotation(R w[3], const R t[3])
{
    const R wt = w[0] * t[0] + w[1] * t[1] + w[2] * t[2];
    const R sf = R(1) / (R(1) + (t[0] * t[0] + t[1] * t[1] + t[2] * t[2]));
    const R x0 = w[1] * t[2] - w[2] * t[1], x1 = w[2] * t[0] - w[0] * t[2], x2 = w[0] * t[1] - w[1] * t[0];
    w[0] = sf * (w[0] + wt * t[0] + x0);
    w[1] = sf * (w[1] + wt * t[1] + x1);
    w[2] = sf * (w[2] + wt * t[2] + x2);
}

// Vay pusher (units of App. C, w = c u): the full electric kick and half
// the magnetic kick with the old velocity, then the other magnetic half with
// the new velocity, solved exactly.
template <typename R>
__device__ __forceinline__ void vay(R u[3], const R e[3], const R b[3], R c, R inv_c, R s)
{
    const R k = R(0.5) * s * inv_c;
    const R tau[3] = {k * b[0], k * b[1], k * b[2]};
    R w[3] = {c * u[0], c * u[1], c * u[2]};
    const R ig0 = R(1) / sqrt(R(1) + u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    const R v[3] = {w[0] * ig0, w[1] * ig0, w[2] * ig0};
    w[0] += s * e[0] + (v[1] * tau[2] - v[2] * tau[1]);
    w[1] += s * e[1] + (v[2] * tau[0] - v[0] * tau[2]);
    w[2] += s * e[2] + (v[0] * tau[1] - v[1] * tau[0]);
    const R ig = R(1) / implicit_gamma<R>(w, tau, inv_c);
    const R t[3] = {tau[0] * ig, tau[1] * ig, tau[2] * ig};
    exact_rotation<R>(w, t);
    u[0] = w[0] * inv_c;
    u[1] = w[1] * inv_c;
    u[2] = w[2] * inv_c;
}

// Higuera-Cary pusher: Boris's split with the rotation's Lorentz factor from
// the implicit relation (volume preserving, exact E x B velocity).
template <typename R>
__device__ __forceinline__ void higuera_cary(R u[3], const R e[3], const R b[3], R c, R inv_c, R s)
{
    const R hs = R(0.5) * s, k = hs * inv_c;
    const R eps[3] = {hs * e[0], hs * e[1], hs * e[2]};
    const R tau[3] = {k * b[0], k * b[1], k * b[2]};
    R w[3] = {c * u[0] + eps[0], c * u[1] + eps[1], c * u[2] + eps[2]};
    const R ig = R(1) / implicit_gamma<R>(w, tau, inv_c);
    const R t[3] = {tau[0] * ig, tau[1] * ig, tau[2] * ig};
    exact_rotation<R>(w, t);
    const R x0 = w[1] * t[2] - w[2] * t[1], x1 = w[2] * t[0] - w[0] * t[2], x2 = w[0] * t[1] - w[1] * t[0];
    u[0] = (w[0] + eps[0] + x0) * inv_c;
    u[1] = (w[1] + eps[1] + x1) * inv_c;
    u[2] = (w[2] + eps[2] + x2) * inv_c;
}

enum : int { PUSHER_BORIS = 0, PUSHER_VAY = 1, PUSHER_HC = 2 };

template <typename R, int PUSHER>
__device__ __forceinline__ void push_u(R u[3], const R e[3], const R b[3], R c, R inv_c, R s)
{
    if constexpr (PUSHER == PUSHER_VAY) vay<R>(u, e, b, c, inv_c, s);
    else if constexpr (PUSHER == PUSHER_HC) higuera_cary<R>(u, e, b, c, inv_c, s);
    else boris<R>(u, e, b, c, inv_c, s);
}

// Eq. (fdX): displacement c u / gamma of u^{n+1/2}, all three components, and
// r = c / gamma, from which end_point forms x + u r in one rounding.  Returns
// gamma^2 = 1 + |u|^2 (finite exactly when u is).  As boris, with the
// multiply-adds written out, so that every kernel puts a particle on the same
// side of a face.
template <typename R>
__device__ __forceinline__ R displacement(const R u[3], R c, R dv[3], R &r)
{
    const R g2 = fma(u[2], u[2], fma(u[1], u[1], fma(u[0], u[0], R(1))));
    r = c * rsqrt_w<R>(g2);
    dv[0] = u[0] * r;
    dv[1] = u[1] * r;
    dv[2] = u[2] * r;
    return g2;
}

template <typename R, int D>
__device__ __forceinline__ void end_point(const R x[3], const R u[3], R r, R x2[3])
{
#pragma unroll
    for (int d = 0; d < D; ++d) x2[d] = fma(u[d], r, x[d]);
}

// ----------------------------------------------------------------- ZigZag

// Current of one straight segment inside one cell, as the values it adds
// to the LDS current block: component m goes to the cell index along m and,
// along each transverse grid dimension a, to points i_a and i_a+1 with
// weights 1-W_a and W_a at the segment midpoint; with two transverse
// dimensions the path average of the product adds
// sigma_a sigma_b dv_a dv_b / 12.  Value order matches seg_offset().
template <int D>
__host__ __device__ constexpr int seg_values()
{
    return D == 1 ? 5 : (D == 2 ? 8 : 12);
}

// The values as flux component times weight: value k is
// F[seg_comp<D>(k)] * wt[k].
template <int D>
__host__ __device__ constexpr int seg_comp(int k)
{
    return D == 1 ? (k == 0 ? 0 : (k < 3 ? 1 : 2)) : (D == 2 ? (k < 2 ? 0 : (k < 4 ? 1 : 2)) : (k < 4 ? 0 : (k < 8 ? 1 : 2)));
}

template <typename R, int D>
__device__ __forceinline__ void segment_weights(const R W[3], const R dv[3], R wt[seg_values<D>()])
{
    if constexpr (D == 1) {
        wt[0] = R(1);
        wt[1] = R(1) - W[0];
        wt[2] = W[0];
        wt[3] = R(1) - W[0];
        wt[4] = W[0];
    } else if constexpr (D == 2) {
        wt[0] = R(1) - W[1];
        wt[1] = W[1];
        wt[2] = R(1) - W[0];
        wt[3] = W[0];
        const R cr = dv[0] * dv[1] * R(1.0 / 12.0);
        wt[4] = (R(1) - W[0]) * (R(1) - W[1]) + cr;
        wt[5] = W[0] * (R(1) - W[1]) - cr;
        wt[6] = (R(1) - W[0]) * W[1] - cr;
        wt[7] = W[0] * W[1] + cr;
    } else {
        const R cyz = dv[1] * dv[2] * R(1.0 / 12.0);
        wt[0] = (R(1) - W[1]) * (R(1) - W[2]) + cyz;
        wt[1] = W[1] * (R(1) - W[2]) - cyz;
        wt[2] = (R(1) - W[1]) * W[2] - cyz;
        wt[3] = W[1] * W[2] + cyz;
        const R cxz = dv[0] * dv[2] * R(1.0 / 12.0);
        wt[4] = (R(1) - W[0]) * (R(1) - W[2]) + cxz;
        wt[5] = W[0] * (R(1) - W[2]) - cxz;
        wt[6] = (R(1) - W[0]) * W[2] - cxz;
        wt[7] = W[0] * W[2] + cxz;
        const R cxy = dv[0] * dv[1] * R(1.0 / 12.0);
        wt[8] = (R(1) - W[0]) * (R(1) - W[1]) + cxy;
        wt[9] = W[0] * (R(1) - W[1]) - cxy;
        wt[10] = (R(1) - W[0]) * W[1] - cxy;
        wt[11] = W[0] * W[1] + cxy;
    }
}

// LDS offsets (relative to the segment's cell) of those values: component
// plane offset plus corner offset.
template <int D>
__device__ __forceinline__ int seg_offset(const Strides st, int k)
{
    const int s1 = st.y, s2 = st.z, n = st.m;
    if constexpr (D == 1) {
        return k == 0 ? 0 : (k == 1 ? n : (k == 2 ? n + 1 : (k == 3 ? 2 * n : 2 * n + 1)));
    } else if constexpr (D == 2) {
        switch (k) {
        case 0: return 0;
        case 1: return s1;
        case 2: return n;
        case 3: return n + 1;
        case 4: return 2 * n;
        case 5: return 2 * n + 1;
        case 6: return 2 * n + s1;
        default: return 2 * n + s1 + 1;
        }
    } else {
        switch (k) {
        case 0: return 0;
        case 1: return s1;
        case 2: return s2;
        case 3: return s1 + s2;
        case 4: return n;
        case 5: return n + 1;
        case 6: return n + s2;
        case 7: return n + 1 + s2;
        case 8: return 2 * n;
        case 9: return 2 * n + 1;
        case 10: return 2 * n + s1;
        default: return 2 * n + s1 + 1;
        }
    }
}

// ZigZag deposit (App. D) of one particle moving from x1 to x2 (tile-local,
// unrebased) with displacement dv (all three components) and charge q.
// Relay point per grid dimension: min(min(i1,i2)+1, max(max(i1,i2),
// (x1+x2)/2)) (App. D); along non-grid dimensions the two segments share dv/2.
// When both segments lie in the same cell they touch the same points, so
// their values are added in registers (F1 w1 + F2 w2, one multiply-add) and
// written with one set of atomics.
// The two cells of a grid dimension differ by at most one, so the relay point
// is the midpoint when they are the same and the larger of the two cell
// indices when not.  st: strides of the block sJ.
template <typename R, int D, typename A>
__device__ __forceinline__ void zigzag(A *sJ, const Strides st, const int32_t T[3], const R x1[3], const R x2[3],
                                       const R dv[3], R q)
{
    R F1[3], F2[3], W1[3] = {0, 0, 0}, W2[3] = {0, 0, 0}, d1[3], d2[3];
    int l1[3] = {0, 0, 0}, l2[3] = {0, 0, 0};
    bool same = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        if (d < D) {
            const R a = x1[d], b = x2[d];
            const R fa = floor(a), fb = floor(b);
            const R xr = fa == fb ? R(0.5) * (a + b) : (fa > fb ? fa : fb);
            d1[d] = xr - a;
            d2[d] = b - xr;
            F1[d] = q * d1[d];
            F2[d] = q * d2[d];
            W1[d] = fma(R(0.5), a + xr, -fa);
            W2[d] = fma(R(0.5), b + xr, -fb);
            l1[d] = (int)fa + T[d] / 2 + 1;
            l2[d] = (int)fb + T[d] / 2 + 1;
            same = same && fa == fb;
        } else {
            R h = R(0.5) * dv[d];
            d1[d] = h;
            d2[d] = h;
            F1[d] = q * h;
            F2[d] = q * h;
        }
    }
    constexpr int NV = seg_values<D>();
    R w1[NV], w2[NV], F2s[3];
    segment_weights<R, D>(W1, d1, w1);
    segment_weights<R, D>(W2, d2, w2);
#pragma unroll
    for (int d = 0; d < 3; ++d) F2s[d] = same ? F2[d] : R(0);
    const int b1 = l1[0] + (D > 1 ? imul24(l1[1], st.y) : 0) + (D > 2 ? imul24(l1[2], st.z) : 0);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int m = seg_comp<D>(k);
        lds_add(sJ + b1 + seg_offset<D>(st, k), fma(F2s[m], w2[k], F1[m] * w1[k]));
    }
    if (!same) {
        const int b2 = l2[0] + (D > 1 ? imul24(l2[1], st.y) : 0) + (D > 2 ? imul24(l2[2], st.z) : 0);
#pragma unroll
        for (int k = 0; k < NV; ++k) lds_add(sJ + b2 + seg_offset<D>(st, k), F2[seg_comp<D>(k)] * w2[k]);
    }
}

// ------------------------------------------------------------------ walls

// Conducting, reflecting walls at x = 0 and x = n0 (y, z periodic): the
// x-staggered components (Ex, By, Bz) see the wall as a mirror, the
// node-centred ones (Ey, Ez, Bx) vanish on the wall plane.  Applied to the
// staged LDS blocks of a wall tile after push_half_b1: the low wall's ghost
// column (local x = -1) and the high wall's column (local x = T) take the
// image values.
template <typename R, int D>
__device__ __forceinline__ void wall_images(R *sF, const CurBox<D> &cb, const FieldBox<D> &fb, const FieldLds<D> &fl,
                                            const int32_t T[3], int walls)
{
    for (int r = threadIdx.x; r < cb.e1 * cb.e2; r += blockDim.x) {
        const int ly = r % cb.e1, lz = r / cb.e1, m = fl.e.m;
        R *E = sF + ly * fl.e.y + lz * fl.e.z;
        if (walls & 1) E[0] = E[1];                             // Ex(-1/2) = Ex(1/2)
        if (walls & 2) {
            E[T[0] + 1] = E[T[0]];                              // Ex(n0+1/2) = Ex(n0-1/2)
            E[m + T[0] + 1] = R(0);                             // Ey, Ez on the wall plane
            E[2 * m + T[0] + 1] = R(0);
        }
    }
    for (int r = threadIdx.x; r < fb.e1 * fb.e2; r += blockDim.x) {
        const int ly = r % fb.e1, lz = r / fb.e1, m = fl.b.m;
        R *B = sF + fl.b0 + ly * fl.b.y + lz * fl.b.z;
        if (walls & 1) {
            B[m] = B[m + 1];                                    // By, Bz mirror
            B[2 * m] = B[2 * m + 1];
        }
        if (walls & 2) {
            B[T[0] + 1] = R(0);                                 // Bx on the wall plane
            B[m + T[0] + 1] = B[m + T[0]];
            B[2 * m + T[0] + 1] = B[2 * m + T[0]];
        }
    }
}

// A particle of a wall tile whose move ends beyond the wall is reflected:
// the current runs along the broken path x1 -> wall point -> mirrored end
// (two ZigZag moves, the non-grid displacement split in proportion), then
// x2 and u_x are mirrored.  Returns false (nothing done) for other moves.
template <typename R, int D, typename A>
__device__ __forceinline__ bool wall_reflect(A *sJ, const Strides st, const int32_t T[3], int walls,
                                             const R x1[3], R x2[3], R u[3], const R dv[3], R q)
{
    const R half = R(T[0] / 2);
    const bool lo = (walls & 1) && x2[0] < -half;
    const bool hi = (walls & 2) && x2[0] >= half;
    if (!(lo || hi)) return false;
    const R wx = lo ? -half : half;
    const R t = (wx - x1[0]) / (x2[0] - x1[0]);
    R w[3] = {wx, 0, 0}, r[3] = {0, 0, 0}, dv1[3] = {0, 0, 0}, dv2[3] = {0, 0, 0};
#pragma unroll
    for (int d = 1; d < 3; ++d) {
        if (d < D) {
            w[d] = x1[d] + t * (x2[d] - x1[d]);
            r[d] = x2[d];
        } else {
            dv1[d] = t * dv[d];
            dv2[d] = dv[d] - dv1[d];
        }
    }
    r[0] = lo ? -R(T[0]) - x2[0] : R(T[0]) - x2[0];
    if (r[0] >= half) r[0] = nextafter(half, R(0));
    zigzag<R, D, A>(sJ, st, T, x1, w, dv1, q);
    zigzag<R, D, A>(sJ, st, T, w, r, dv2, q);
#pragma unroll
    for (int d = 0; d < D; ++d) x2[d] = r[d];
    u[0] = -u[0];
    return true;
}

template <int D>
__host__ __device__ constexpr int centre_code()
{
    return D == 1 ? 1 : (D == 2 ? 4 : 13);
}

// Tile offset code sum (delta_d+1) 3^d of a position after the push.
template <typename R, int D>
__device__ __forceinline__ int direction_code(const R x[3], const int32_t T[3], int delta[3])
{
    int code = 0, p3 = 1;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        R half = R(T[d] / 2);
        delta[d] = x[d] < -half ? -1 : (x[d] >= half ? 1 : 0);
        code += (delta[d] + 1) * p3;
        p3 *= 3;
    }
    return code;
}

// The same code, and the position rebased by -delta T, without comparisons
// per face: the tile offset of the cell floor(x) is floor((cell + T/2) / T),
// and (cell + T/2 + 1/2) / T stays 1/(2T) away from an integer, more than the
// rounding of the product with 1/T.  Exact for any even T below 2^20.
template <typename R, int D>
__device__ __forceinline__ int rebase(const R x[3], const int32_t T[3], R xr[3])
{
    R code = R(0);
#pragma unroll
    for (int d = D - 1; d >= 0; --d) {
        const R inv = R(1) / R(T[d]);
        const R delta = floor(fma(floor(x[d]), inv, R(0.5) + R(0.5) * inv));
        xr[d] = fma(-R(T[d]), delta, x[d]);
        code = fma(code, R(3), delta);
    }
    return (int)code + centre_code<D>();
}

template <int D>
__host__ __device__ constexpr int ncodes()
{
    return D == 1 ? 3 : (D == 2 ? 9 : 27);
}

}  // namespace pic
