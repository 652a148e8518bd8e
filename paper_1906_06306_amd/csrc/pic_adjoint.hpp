// Adjoint (reverse mode) of the fused step on gfx950: the vector-Jacobian
// product of one step, for gradients of a loss of a later state with respect
// to an earlier one (differentiable windows with checkpointed recomputation).
//
// The per-particle part mirrors the push: one work-group per tile stages E,
// B (then B^n in LDS) and the current adjoint lambda_J with their halos,
// recomputes each particle's push, and runs it backwards: ZigZag adjoint
// (derivatives of its segment values), position and displacement adjoints,
// Boris adjoint (hand-derived reverse of App. C) and the interpolation adjoint, whose scatter into the
// field adjoints goes to FP64 LDS blocks that are flushed and folded like the
// current.
#pragma once

#include "pic_kernels.hpp"

namespace pic {

// ------------------------------------------------------ ZigZag adjoint

// Value j of one component of a straight segment (segment_weights) is F w; its
// derivatives are dF w along the component and F da, F db along the NT
// transverse grid dimensions a (and b).  i = 0, 1: with respect to x1, x2.
template <typename R, int NT>
struct SegmentGrad {
    R Wa, Wb, ma, mb, c, dWa[2], dWb[2], ca[2], cb[2];
    R w, da[2], db[2];
    __device__ __forceinline__ SegmentGrad(const R W[3], const R d[3], const R dW[3][2], const R dd[3][2], int a, int b)
    {
#pragma clang fp contract(off)
        if constexpr (NT > 0) {
            Wa = W[a];
            ma = R(1) - Wa;
            dWa[0] = dW[a][0];
            dWa[1] = dW[a][1];
        }
        if constexpr (NT > 1) {
            Wb = W[b];
            mb = R(1) - Wb;
            dWb[0] = dW[b][0];
            dWb[1] = dW[b][1];
            const R k = R(1.0 / 12.0);
            c = d[a] * d[b] * k;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                ca[i] = dd[a][i] * d[b] * k;
                cb[i] = d[a] * dd[b][i] * k;
            }
        }
    }
    __device__ __forceinline__ void value(int j)
    {
#pragma clang fp contract(off)
        const bool ja = j & 1, jb = j & 2;
        if constexpr (NT == 0) {
            w = R(1);
        } else if constexpr (NT == 1) {
            w = ja ? Wa : ma;
            da[0] = ja ? dWa[0] : -dWa[0];
            da[1] = ja ? dWa[1] : -dWa[1];
        } else {
            const R wa = ja ? Wa : ma, wb = jb ? Wb : mb;
            const bool plus = ja == jb;
            w = fma(wa, wb, plus ? c : -c);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                da[i] = (ja ? dWa[i] : -dWa[i]) * wb + (plus ? ca[i] : -ca[i]);
                db[i] = wa * (jb ? dWb[i] : -dWb[i]) + (plus ? cb[i] : -cb[i]);
            }
        }
    }
};

// d(sum_points lambda_J . J)/d(x1, x2, dv_nongrid) of one particle's ZigZag
// deposit.  The relay point and cells are taken on the branch of the forward
// value; sLJ is the staged lambda_J block (local cells -1..T+1).  Derivatives
// run forward through the segment values, two ends per grid dimension, with
// the products that are zero for every particle left out (dual numbers of
// 2D + (3 - D) parts: 1,545 vector instructions per 64 particles of the 2D FP32
// kernel, 193 registers, 186 us per step of a shear layer of 256^2 cells, 32
// particles each; this: 1,125, 110 and 142 us).  Multiply-adds are written out and
// nothing else is contracted: in 1D and 2D the results are those of the dual
// numbers, bit for bit, in 3D FP32 as near to the FP64 ones (2.50e-7 relative
// for the position adjoints of 32x32x24 cells with either).
template <typename R, int D, typename LA>
__device__ __forceinline__ void zigzag_adjoint(const LA *sLJ, const Strides st, const int32_t T[3], const R x1[3],
                                               const R x2[3], const R dv[3], R q, R lx1[3], R lx2[3], R ldv[3])
{
#pragma clang fp contract(off)
    R F[2][3], W[2][3], d[2][3], dF[2][3][2], dW[2][3][2], dd[2][3][2];
    int base[2] = {0, 0};
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        if (m < D) {
            const R a = x1[m], b = x2[m];
            const R fa = floor(a), fb = floor(b);
            // the relay point is the midpoint (also where that lies on the
            // face), else the face between the cells
            const R half = R(0.5) * (a + b), face = fa > fb ? fa : fb;
            const bool mid = fa == fb || half == face;
            const R xr = mid ? half : face, h = mid ? R(0.5) : R(0);   // h: d xr / d x1 = d xr / d x2
            d[0][m] = xr - a;
            d[1][m] = b - xr;
            dd[0][m][0] = h - R(1);
            dd[0][m][1] = h;
            dd[1][m][0] = -h;
            dd[1][m][1] = R(1) - h;
            W[0][m] = R(0.5) * (a + xr) - fa;
            W[1][m] = R(0.5) * (b + xr) - fb;
            dW[0][m][0] = dW[1][m][1] = R(0.5) * (R(1) + h);
            dW[0][m][1] = dW[1][m][0] = R(0.5) * h;
            const int sm = m == 0 ? 1 : (m == 1 ? st.y : st.z);
            base[0] += imul24((int)fa + T[m] / 2 + 1, sm);
            base[1] += imul24((int)fb + T[m] / 2 + 1, sm);
        } else {
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                d[g][m] = R(0.5) * dv[m];
                dd[g][m][0] = R(0.5);
                dd[g][m][1] = R(0);
            }
        }
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            F[g][m] = q * d[g][m];
#pragma unroll
            for (int i = 0; i < 2; ++i) dF[g][m][i] = q * dd[g][m][i];
        }
    }
    R lin[3][2] = {};
    auto component = [&](auto nt, int m, int a, int b, int v0) {
#pragma clang fp contract(off)
        constexpr int NT = decltype(nt)::value;
        SegmentGrad<R, NT> s0(W[0], d[0], dW[0], dd[0], a, b), s1(W[1], d[1], dW[1], dd[1], a, b);
#pragma unroll
        for (int j = 0; j < (1 << NT); ++j) {
            s0.value(j);
            s1.value(j);
            const R la = (R)sLJ[base[0] + seg_offset<D>(st, v0 + j)];
            const R lb = (R)sLJ[base[1] + seg_offset<D>(st, v0 + j)];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (m < D || i == 0) lin[m][i] = lin[m][i] + fma(la, dF[0][m][i] * s0.w, lb * (dF[1][m][i] * s1.w));
                if constexpr (NT > 0)
                    lin[a][i] = lin[a][i] + fma(la, F[0][m] * s0.da[i], lb * (F[1][m] * s1.da[i]));
                if constexpr (NT > 1)
                    lin[b][i] = lin[b][i] + fma(la, F[0][m] * s0.db[i], lb * (F[1][m] * s1.db[i]));
            }
            __builtin_amdgcn_sched_barrier(0);   // one value at a time: fewer registers
        }
    };
    using N0 = std::integral_constant<int, 0>;
    using N1 = std::integral_constant<int, 1>;
    using N2 = std::integral_constant<int, 2>;
    if constexpr (D == 1) {
        component(N0(), 0, 0, 0, 0);
        component(N1(), 1, 0, 0, 1);
        component(N1(), 2, 0, 0, 3);
    } else if constexpr (D == 2) {
        component(N1(), 0, 1, 0, 0);
        component(N1(), 1, 0, 0, 2);
        component(N2(), 2, 0, 1, 4);
    } else {
        component(N2(), 0, 1, 2, 0);
        component(N2(), 1, 0, 2, 4);
        component(N2(), 2, 0, 1, 8);
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        if (m < D) {
            lx1[m] += lin[m][0];
            lx2[m] += lin[m][1];
        } else {
            ldv[m] += lin[m][0];
        }
    }
}

// --------------------------------------------------- interpolation adjoint

// Value, gradient with respect to the particle position, and (with SCATTER)
// the scatter lam * weight into the FP64 adjoint block L of one
// staggered component (same stencil as interp_at).
template <typename R, int D, int COMP, bool SCATTER>
__device__ __forceinline__ R interp_comp_adj(const R *__restrict__ F, double *L, int s1, int s2,
                                             const Stencil<R, D> &st, R lam, R g[3])
{
    constexpr bool h0 = COMP == 0 || COMP == 4 || COMP == 5;
    constexpr bool h1 = COMP == 1 || COMP == 3 || COMP == 5;
    constexpr bool h2 = COMP == 2 || COMP == 3 || COMP == 4;
    int b = h0 ? st.bh[0] : st.bn[0];
    const R w0 = h0 ? st.wh[0] : st.wn[0];
    if constexpr (D == 1) {
        g[0] = F[b + 1] - F[b];
        if constexpr (SCATTER) {
            lds_add(L + b, lam * (R(1) - w0));
            lds_add(L + b + 1, lam * w0);
        }
        return F[b] * (R(1) - w0) + F[b + 1] * w0;
    } else if constexpr (D == 2) {
        b += (h1 ? st.bh[1] : st.bn[1]) * s1;
        const R w1 = h1 ? st.wh[1] : st.wn[1];
        const R f00 = F[b], f10 = F[b + 1], f01 = F[b + s1], f11 = F[b + s1 + 1];
        const R a0 = f00 * (R(1) - w0) + f10 * w0, a1 = f01 * (R(1) - w0) + f11 * w0;
        g[0] = (f10 - f00) * (R(1) - w1) + (f11 - f01) * w1;
        g[1] = a1 - a0;
        if constexpr (SCATTER) {
            lds_add(L + b, lam * (R(1) - w0) * (R(1) - w1));
            lds_add(L + b + 1, lam * w0 * (R(1) - w1));
            lds_add(L + b + s1, lam * (R(1) - w0) * w1);
            lds_add(L + b + s1 + 1, lam * w0 * w1);
        }
        return a0 * (R(1) - w1) + a1 * w1;
    } else {
        b += (h1 ? st.bh[1] : st.bn[1]) * s1;
        b += (h2 ? st.bh[2] : st.bn[2]) * s2;
        const R w1 = h1 ? st.wh[1] : st.wn[1];
        const R w2 = h2 ? st.wh[2] : st.wn[2];
        R f[8];
#pragma unroll
        for (int cn = 0; cn < 8; ++cn) f[cn] = F[b + (cn & 1) + ((cn >> 1) & 1) * s1 + ((cn >> 2) & 1) * s2];
        R val = R(0);
        g[0] = g[1] = g[2] = R(0);
#pragma unroll
        for (int cn = 0; cn < 8; ++cn) {
            const int c0 = cn & 1, c1 = (cn >> 1) & 1, c2 = (cn >> 2) & 1;
            const R p0 = c0 ? w0 : R(1) - w0, p1 = c1 ? w1 : R(1) - w1, p2 = c2 ? w2 : R(1) - w2;
            val += f[cn] * p0 * p1 * p2;
            g[0] += f[cn] * (c0 ? R(1) : R(-1)) * p1 * p2;
            g[1] += f[cn] * p0 * (c1 ? R(1) : R(-1)) * p2;
            g[2] += f[cn] * p0 * p1 * (c2 ? R(1) : R(-1));
            if constexpr (SCATTER) lds_add(L + b + c0 + c1 * s1 + c2 * s2, lam * p0 * p1 * p2);
        }
        return val;
    }
}

// ------------------------------------------------------------ Boris adjoint

// Reverse of boris(): from u0 = u^{n-1/2}, the fields at the particle and
// lu1 = lambda of u^{n+1/2}, the adjoints of u0, E and B.  Written from the
// exact update (division and square root), independent of how the forward
// evaluates them.
template <typename R>
__device__ __forceinline__ void boris_adjoint(const R u0[3], const R e[3], const R bf[3], R c, R inv_c, R s,
                                              const R lu1[3], R lu0[3], R lE[3], R lB[3])
{
    const R hs = R(0.5) * s;
    R eps[3], a[3], t[3], w[3], b[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        eps[i] = hs * e[i];
        a[i] = c * u0[i] + eps[i];
    }
    const R g1 = sqrt(R(1) + (a[0] * a[0] + a[1] * a[1] + a[2] * a[2]) * (inv_c * inv_c));
    const R kap = hs * inv_c / g1;
#pragma unroll
    for (int i = 0; i < 3; ++i) t[i] = kap * bf[i];
    const R f = R(2) / (R(1) + (t[0] * t[0] + t[1] * t[1] + t[2] * t[2]));
    w[0] = a[0] + (a[1] * t[2] - a[2] * t[1]);
    w[1] = a[1] + (a[2] * t[0] - a[0] * t[2]);
    w[2] = a[2] + (a[0] * t[1] - a[1] * t[0]);
#pragma unroll
    for (int i = 0; i < 3; ++i) b[i] = f * w[i];
    R lc[3], la[3], leps[3], lb[3], lt[3], lw[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lc[i] = lu1[i] * inv_c;
        la[i] = lc[i];
        leps[i] = lc[i];
    }
    lb[0] = t[1] * lc[2] - t[2] * lc[1];
    lb[1] = t[2] * lc[0] - t[0] * lc[2];
    lb[2] = t[0] * lc[1] - t[1] * lc[0];
    lt[0] = lc[1] * b[2] - lc[2] * b[1];
    lt[1] = lc[2] * b[0] - lc[0] * b[2];
    lt[2] = lc[0] * b[1] - lc[1] * b[0];
    R lf = R(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lw[i] = f * lb[i];
        lf += w[i] * lb[i];
    }
    la[0] += lw[0] + (t[1] * lw[2] - t[2] * lw[1]);
    la[1] += lw[1] + (t[2] * lw[0] - t[0] * lw[2]);
    la[2] += lw[2] + (t[0] * lw[1] - t[1] * lw[0]);
    lt[0] += lw[1] * a[2] - lw[2] * a[1];
    lt[1] += lw[2] * a[0] - lw[0] * a[2];
    lt[2] += lw[0] * a[1] - lw[1] * a[0];
#pragma unroll
    for (int i = 0; i < 3; ++i) lt[i] -= lf * f * f * t[i];
    R lkap = R(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lB[i] = kap * lt[i];
        lkap += bf[i] * lt[i];
    }
    const R lg1 = -kap / g1 * lkap;
#pragma unroll
    for (int i = 0; i < 3; ++i) la[i] += lg1 * a[i] * (inv_c * inv_c) / g1;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        lu0[i] = c * la[i];
        leps[i] += la[i];
        lE[i] = hs * leps[i];
    }
}

// ------------------------------------------------------------ kernels

template <typename R>
struct AdjParams {
    R *lpos, *lu;             // [D|3][cap_total], layout of the state
    R *lE, *lB;               // [3][cells_total]
    R *lJ;                    // [3][cells_total] scratch: lambda_B between the two halves of k_adj_fields
    R *eblk, *bblk;           // per tile [3][(T+3)^D], [3][(T+2)^D] adjoint blocks
    R *opos, *ou;             // [D|3][ostride] particle adjoints at the slots the particles
    int64_t ostride;          // came from (Params::ids), or null: in place
};

// Threads of k_adj_push: 512 (16 waves per CU at the shear window's 1,024
// tiles of 8^2) where its registers allow them without spilling.
template <typename R, int D>
__host__ __device__ constexpr int adj_block()
{
    return sizeof(R) == 4 && D < 3 ? 512 : 256;
}

// Per tile: the particle part of the adjoint step.  State in p (particles
// x^n, u^{n-1/2}; E^n, B^{n-1/2}); on entry a.lpos/a.lu hold the adjoints of
// x^{n+1}, u^{n+1/2} (same slots), on exit those of x^n, u^{n-1/2}; the
// interpolation adjoints go to the per-tile blocks a.eblk (for E^n) and
// a.bblk (for B^n).
template <typename R, int D, int TC>
__global__ void __launch_bounds__((adj_block<R, D>())) k_adj_push(Params<R> p, AdjParams<R> a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int t = blockIdx.x;
    const TileDesc td = p.tiles[t];
    // tile edge: a compile-time constant when TC > 0, as in the push
    const int32_t T[3] = {TC > 0 ? TC : p.T[0], D > 1 ? (TC > 0 ? TC : p.T[1]) : 1, D > 2 ? (TC > 0 ? TC : p.T[2]) : 1};
    const FieldBox<D> fb(T);
    const CurBox<D> cb(T);
    double *aE = reinterpret_cast<double *>(smem);           // [3][cb.n]
    double *aB = aE + 3 * cb.n;                              // [3][fb.n]
    R *sLJ = reinterpret_cast<R *>(aB + 3 * fb.n);           // [3][cb.n]
    R *sE = sLJ + 3 * cb.n;                                  // [3][cb.n]
    R *sB = sE + 3 * cb.n;                                   // [3][fb.n]
    stage_block<R, D>(p.E, p.cells_total, td, T, sE, cb);
    stage_block<R, D>(p.B, p.cells_total, td, T, sB, fb);
    // add_cur: E^{n+1} = ... - J, so lambda_J = -lambda_E
    stage_block<R, D, true>(a.lE, p.cells_total, td, T, sLJ, cb);
    for (int k = threadIdx.x; k < 3 * cb.n; k += blockDim.x) aE[k] = 0.0;
    for (int k = threadIdx.x; k < 3 * fb.n; k += blockDim.x) aB[k] = 0.0;
    __syncthreads();
    half_b_lds<R, D>(sB, fb.planes(), fb, sE, cb.planes(), R(0.5) * p.c, td, T, nullptr, 0);   // B^n, as the push saw it
    __syncthreads();
    const R c = p.c, inv_c = p.inv_c;
    const int64_t cap = p.cap_total;
    const int e1 = cb.e0, e2 = cb.e0 * cb.e1, f1 = fb.e0, f2 = fb.e0 * fb.e1;
    for (int s = 0; s < p.nspecies; ++s) {
        const int ts = t * p.nspecies + s;
        const int64_t so = uniform(p.seg_off[ts]);
        const int cnt = uniform(p.seg_cnt[ts]);
        const R q = uniform(p.charge[td.box * p.nspecies + s]);
        const R sq = uniform(p.qm[td.box * p.nspecies + s]);
        for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
            R x[3] = {0, 0, 0}, u0[3], lx[3] = {0, 0, 0}, lu[3];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                x[d] = p.pos[d * cap + so + i];
                lx[d] = a.lpos[d * cap + so + i];
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                u0[m] = p.u[m * cap + so + i];
                lu[m] = a.lu[m * cap + so + i];
            }
            // where the adjoint goes: the particle's own slot, or the one it
            // came from in the step before (its state's origin ids), which
            // saves a pass over the adjoints per reversed step
            int64_t dst = so + i, stride = cap;
            R *opos = a.lpos, *ou = a.lu;
            if (a.opos) {
                dst = p.ids[so + i];
                stride = a.ostride;
                opos = a.opos;
                ou = a.ou;
                if (dst < 0 || dst >= stride) {
                    latch(p.err, ERR_ADJ_MAP);
                    continue;
                }
            }
            auto store = [&](const R px[3], const R pu[3]) {
#pragma unroll
                for (int d = 0; d < D; ++d) opos[d * stride + dst] = px[d];
#pragma unroll
                for (int m = 0; m < 3; ++m) ou[m * stride + dst] = pu[m];
            };
            if (!inside_tile<R, D>(x, T)) {
                if (a.opos) store(lx, lu);
                continue;
            }
            // forward recomputation of this particle's push
            Stencil<R, D> st;
            make_stencil<R, D>(x, T, st);
            R e[3], b[3], g[6][3];
            e[0] = interp_comp_adj<R, D, 0, false>(sE + 0 * cb.n, nullptr, e1, e2, st, R(0), g[0]);
            e[1] = interp_comp_adj<R, D, 1, false>(sE + 1 * cb.n, nullptr, e1, e2, st, R(0), g[1]);
            e[2] = interp_comp_adj<R, D, 2, false>(sE + 2 * cb.n, nullptr, e1, e2, st, R(0), g[2]);
            b[0] = interp_comp_adj<R, D, 3, false>(sB + 0 * fb.n, nullptr, f1, f2, st, R(0), g[3]);
            b[1] = interp_comp_adj<R, D, 4, false>(sB + 1 * fb.n, nullptr, f1, f2, st, R(0), g[4]);
            b[2] = interp_comp_adj<R, D, 5, false>(sB + 2 * fb.n, nullptr, f1, f2, st, R(0), g[5]);
            R u1[3] = {u0[0], u0[1], u0[2]}, dv[3], x2[3] = {0, 0, 0};
            boris<R>(u1, e, b, c, inv_c, sq);
            R r;
            displacement<R>(u1, c, dv, r);
            end_point<R, D>(x, u1, r, x2);
            if (!(finite3<R>(u1) && moved_ok<R, D>(x2, dv, T))) {
                if (a.opos) store(lx, lu);
                continue;
            }
            __builtin_amdgcn_sched_barrier(0);
            // reverse: comp_curr
            R ldv[3] = {0, 0, 0}, lx1[3] = {0, 0, 0};
            zigzag_adjoint<R, D, R>(sLJ, cb.planes(), T, x, x2, dv, q, lx1, lx, ldv);
            // x2 = x + dv
#pragma unroll
            for (int d = 0; d < D; ++d) {
                lx1[d] += lx[d];
                ldv[d] += lx[d];
            }
            // dv = c u1 / gamma(u1)
            const R gam = sqrt(R(1) + u1[0] * u1[0] + u1[1] * u1[1] + u1[2] * u1[2]);
            const R ul = u1[0] * ldv[0] + u1[1] * ldv[1] + u1[2] * ldv[2];
#pragma unroll
            for (int m = 0; m < 3; ++m) lu[m] += c * (ldv[m] / gam - u1[m] * ul / (gam * gam * gam));
            // Boris
            R lu0[3], lEp[3], lBp[3];
            boris_adjoint<R>(u0, e, b, c, inv_c, sq, lu, lu0, lEp, lBp);
            // interpolation: scatter into the field adjoints, gradient in x
            R gg[3];
            interp_comp_adj<R, D, 0, true>(sE + 0 * cb.n, aE + 0 * cb.n, e1, e2, st, lEp[0], gg);
            interp_comp_adj<R, D, 1, true>(sE + 1 * cb.n, aE + 1 * cb.n, e1, e2, st, lEp[1], gg);
            interp_comp_adj<R, D, 2, true>(sE + 2 * cb.n, aE + 2 * cb.n, e1, e2, st, lEp[2], gg);
            interp_comp_adj<R, D, 3, true>(sB + 0 * fb.n, aB + 0 * fb.n, f1, f2, st, lBp[0], gg);
            interp_comp_adj<R, D, 4, true>(sB + 1 * fb.n, aB + 1 * fb.n, f1, f2, st, lBp[1], gg);
            interp_comp_adj<R, D, 5, true>(sB + 2 * fb.n, aB + 2 * fb.n, f1, f2, st, lBp[2], gg);
#pragma unroll
            for (int d = 0; d < D; ++d)
                lx1[d] += lEp[0] * g[0][d] + lEp[1] * g[1][d] + lEp[2] * g[2][d] + lBp[0] * g[3][d] +
                          lBp[1] * g[4][d] + lBp[2] * g[5][d];
            store(lx1, lu0);
        }
    }
    __syncthreads();
    R *eb = a.eblk + (int64_t)t * 3 * cb.n;
    R *bb = a.bblk + (int64_t)t * 3 * fb.n;
    for (int k = threadIdx.x; k < 3 * cb.n; k += blockDim.x) eb[k] = (R)aE[k];
    for (int k = threadIdx.x; k < 3 * fb.n; k += blockDim.x) bb[k] = (R)aB[k];
}

// Sum over the neighbours' blocks of the adjoint entries of component m at the
// tile's cell l: blocks of edges T + HI per dimension from local cell -1 (E:
// HI = 3, B: HI = 2).
template <typename R, int D, int HI>
__device__ __forceinline__ R adj_block_sum(const R *blk, const TileDesc &td, const int32_t T[3], const int l[3], int m)
{
    const int e0 = T[0] + HI, e1 = D > 1 ? T[1] + HI : 1, n = e0 * e1 * (D > 2 ? T[2] + HI : 1);
    R acc = R(0);
#pragma unroll
    for (int oz = (D > 2 ? -1 : 0); oz <= (D > 2 ? 1 : 0); ++oz)
#pragma unroll
        for (int oy = (D > 1 ? -1 : 0); oy <= (D > 1 ? 1 : 0); ++oy)
#pragma unroll
            for (int ox = -1; ox <= 1; ++ox) {
                const int o[3] = {ox, oy, oz};
                int bi[3] = {0, 0, 0}, nc[3] = {0, 0, 0};
                bool in = true;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    bi[d] = l[d] - o[d] * T[d] + 1;
                    in = in && bi[d] >= 0 && bi[d] < T[d] + HI;
                    nc[d] = wrap_once(td.tc[d] + o[d], td.nt[d]);
                }
                const int64_t nid = td.tile0 + nc[0] + td.nt[0] * (nc[1] + (int64_t)td.nt[1] * nc[2]);
                if (in) acc += blk[(nid * 3 + m) * n + bi[0] + e0 * (bi[1] + e1 * bi[2])];
            }
    return acc;
}

// The field rows of the reversed step, from its end, after k_adj_push (which
// reads lambda_E as it enters the step).  Two launches in place of five: each
// is one or two memory latencies, a launch costs as much (a step of the 256^2
// shear layer: 31 us in five launches, 12 us in two).
//
// FIRST: push_e, E^{n+1} = E^n + c curl- B^{n+1/2}: lambda_B += c curl+
// lambda_E, kept in lJ for the other launch; then the particles' part of
// lambda_B.
// Second: push_half_b2 and push_half_b1, B -= (c/2) curl+ E^n: lambda_E -= (c/2)
// curl- lambda_B with lambda_B before and after the particles' part, which for
// lambda_E comes in between.
// One thread per cell and component.
template <typename R, int D, bool FIRST>
__global__ void __launch_bounds__(256) k_adj_fields(Params<R> p, AdjParams<R> a)
{
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const TileDesc td = p.tiles[t];
    const int32_t T[3] = {p.T[0], D > 1 ? p.T[1] : 1, D > 2 ? p.T[2] : 1};
    const int ncell = T[0] * T[1] * T[2];
    const float inv0 = 1.0f / T[0], inv1 = 1.0f / T[1], invc = 1.0f / ncell;
    const int64_t N = p.cells_total;
    const R h = R(-0.5) * p.c;
    for (int k = threadIdx.x; k < 3 * ncell; k += blockDim.x) {
        const int m = div_small(k, invc);
        int l[3];
        cell_of<D>(k - m * ncell, T[0], T[1], inv0, inv1, l[0], l[1], l[2]);
        const int i = m == 2 ? 0 : m + 1, j = m == 0 ? 2 : m - 1;   // curl_m F = d_i F_j - d_j F_i
        int g3[3] = {0, 0, 0};
#pragma unroll
        for (int d = 0; d < D; ++d) g3[d] = td.tc[d] * T[d] + l[d];
        auto at = [&](int axis, int o) -> int64_t {
            const int x = axis == 0 ? wrap_once(g3[0] + o, td.n[0]) : g3[0];
            const int y = D > 1 && axis == 1 ? wrap_once(g3[1] + o, td.n[1]) : g3[1];
            const int z = D > 2 && axis == 2 ? wrap_once(g3[2] + o, td.n[2]) : g3[2];
            return td.cell0 + x + (int64_t)td.n[0] * (y + (int64_t)td.n[1] * z);
        };
        const int64_t g = at(0, 0);
        // neighbours along i and j; the cell itself along axes that are no grid dimension
        const int64_t gi = at(i, FIRST ? 1 : -1), gj = at(j, FIRST ? 1 : -1);
        if constexpr (FIRST) {
            const R *Fi = a.lE + i * N, *Fj = a.lE + j * N;
            const R curl = (Fj[gi] - Fj[g]) - (Fi[gj] - Fi[g]);
            const R b = fma(p.c, curl, a.lB[m * N + g]);
            a.lJ[m * N + g] = b;
            a.lB[m * N + g] = b + adj_block_sum<R, D, 2>(a.bblk, td, T, l, m);
        } else {
            auto curl = [&](const R *F) -> R {
                const R *Fi = F + i * N, *Fj = F + j * N;
                return (Fj[g] - Fj[gi]) - (Fi[g] - Fi[gj]);
            };
            const R e = fma(h, curl(a.lJ), a.lE[m * N + g]) + adj_block_sum<R, D, 3>(a.eblk, td, T, l, m);
            a.lE[m * N + g] = fma(h, curl(a.lB), e);
        }
    }
}

// The state regions that a reversed window keeps of every step, in the
// workspace or in a state image.
template <typename R>
struct StateView {
    R *E, *B, *pos, *u;
    int32_t *seg_cnt, *err, *nf_seg, *ids;
};

// Copy a state: fields, counts, the error word, and of the particle planes
// the slots in use (planes have room for the densest the plasma gets: copying
// them whole moved 2.1 times the bytes on the shear window).  The first
// work-groups take a segment each, 16 (32 at FP64) bytes a lane; the rest
// the fields.  With merge the source's error bits are added to the
// destination's: a load clears none that was latched since.
template <typename R, int D>
__global__ void __launch_bounds__(256) k_state_copy(StateView<R> dst, StateView<R> src, const int64_t *seg_off,
                                                    int32_t nseg, int64_t cap, int64_t cells, int32_t merge)
{
    // vector types: the compiler kept an array of structs of four in private
    // memory and LDS (4.2 million particles of 256^2 cells, FP32 40 us and 33 us
    // without, 6.2 TB/s; FP64 101 and 77 us)
    typedef R Quad __attribute__((ext_vector_type(4)));
    typedef int32_t Quad4 __attribute__((ext_vector_type(4)));
    if ((int)blockIdx.x >= nseg) {
        const int64_t step = (int64_t)(gridDim.x - nseg) * blockDim.x;
        for (int64_t i = (int64_t)(blockIdx.x - nseg) * blockDim.x + threadIdx.x; i < 3 * cells; i += step) {
            const R e = src.E[i], b = src.B[i];
            dst.E[i] = e;
            dst.B[i] = b;
        }
        if ((int)blockIdx.x == nseg && threadIdx.x == 0) {
            if (merge) latch(dst.err, *src.err);
            else *dst.err = *src.err;
        }
        return;
    }
    const int ts = blockIdx.x;
    const int64_t so = seg_off[ts];
    const int cnt = src.seg_cnt[ts];
    if (threadIdx.x == 0) {
        dst.seg_cnt[ts] = cnt;
        dst.nf_seg[ts] = src.nf_seg[ts];
    }
    // segments start at multiples of 64 slots and hold a multiple of 64
    for (int i = threadIdx.x * 4; i < cnt; i += blockDim.x * 4) {
        Quad v[D + 3];
#pragma unroll
        for (int d = 0; d < D; ++d) v[d] = *reinterpret_cast<const Quad *>(src.pos + d * cap + so + i);
#pragma unroll
        for (int m = 0; m < 3; ++m) v[D + m] = *reinterpret_cast<const Quad *>(src.u + m * cap + so + i);
        const Quad4 id = *reinterpret_cast<const Quad4 *>(src.ids + so + i);
#pragma unroll
        for (int d = 0; d < D; ++d) *reinterpret_cast<Quad *>(dst.pos + d * cap + so + i) = v[d];
#pragma unroll
        for (int m = 0; m < 3; ++m) *reinterpret_cast<Quad *>(dst.u + m * cap + so + i) = v[D + m];
        *reinterpret_cast<Quad4 *>(dst.ids + so + i) = id;
    }
}

// Move particle adjoints from the slots of the current state to the slots
// (or input indices) the particles came from: dst = ids[j].  Grid: x over
// (tile, species) segments, y over chunks of blockDim slots of a segment.
template <typename R, int D>
__global__ void __launch_bounds__(256) k_adj_unpermute(Params<R> p, const R *lpos_a, const R *lu_a, R *lpos_b,
                                                       R *lu_b, int64_t stride_b)
{
    const int ts = blockIdx.x;
    const int j = blockIdx.y * blockDim.x + threadIdx.x;
    const int cnt = p.seg_cnt[ts];
    if (j >= cnt) return;
    const int64_t cap = p.cap_total;
    const int64_t src = p.seg_off[ts] + j, dst = p.ids[src];
    if (dst < 0 || dst >= stride_b) {
        latch(p.err, ERR_ADJ_MAP);
        return;
    }
#pragma unroll
    for (int d = 0; d < D; ++d) lpos_b[d * stride_b + dst] = lpos_a[d * cap + src];
#pragma unroll
    for (int m = 0; m < 3; ++m) lu_b[m * stride_b + dst] = lu_a[m * cap + src];
}

}  // namespace pic
