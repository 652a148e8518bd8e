// Kernels of the relativistic PIC step for gfx950 (templated on precision
// R and dimension D).  One work-group owns one tile: it stages the tile's
// E and B (plus halo) in LDS, streams the tile's particles with coalesced
// structure-of-arrays loads, accumulates the ZigZag current in an LDS block
// with atomics and flushes that block once.  Field kernels also walk tiles.
#pragma once

#include "pic_device.hpp"

namespace pic {

constexpr int MAX_WAVES = 16;

// Inclusive prefix sum of v over each row of 16 lanes (DPP row shifts; a
// shifted-in lane outside the row reads 0).  Lanes 0..15 hold the prefix of
// lanes 0..15.
__device__ __forceinline__ int row_prefix16(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    return v;
}

// The per-wave totals of a work-group scan (written by lane 0 of every wave
// to tot[wave], before a barrier; the entries past the wave count are zero):
// returns the sum over the waves below this one and, in all, over every wave.
// Lane w reads the total of wave w and the first 16 lanes scan them, so the
// cost does not grow with the wave count.
__device__ __forceinline__ int wave_totals(const int *tot, int wave, int nw, int &all)
{
    const int lane = threadIdx.x & 63;
    const int v = tot[lane & (MAX_WAVES - 1)];
    const int incl = row_prefix16(v);
    all = __builtin_amdgcn_readlane(incl, nw - 1);
    return __builtin_amdgcn_readlane(incl - v, wave);
}

// Exclusive prefix of a per-thread flag over the whole work-group (wave
// ballots, then per-wave totals in LDS).  sTot holds 2*MAX_WAVES ints, zero
// before the first call, and the two halves alternate by `parity`, so one
// barrier per call suffices.
__device__ __forceinline__ int wg_scan_flag(bool flag, int *sTot, int parity, int &total)
{
    const int lane = threadIdx.x & 63;
    // the wave index and wave count are uniform (scalar registers)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
    const unsigned long long m = __builtin_amdgcn_ballot_w64(flag);
    int below = lanes_below(m);
    int *tot = sTot + parity * MAX_WAVES;
    if (lane == 0) tot[wave] = __popcll(m);
    __syncthreads();
    const int off = wave_totals(tot, wave, nw, total);
    return off + below;
}

// LDS of bucket_outbox, in ints: the histogram of the codes, which becomes
// the bucket starts, and per-wave code counts.
template <int D>
__host__ __device__ constexpr int bucket_lds_ints()
{
    return ncodes<D>() + 1 + MAX_WAVES * ncodes<D>();
}

// Stable counting sort of one segment's n outbox entries by direction code:
// the bucket starts ob_boff[ncodes + 1] and the outbox slots in bucket order
// ob_idx, so that each neighbour reads exactly the leavers addressed to it.
// code_of(k) is the code of entry k; sBase holds the histogram of the codes
// (complete before a barrier) and receives the bucket starts.  The rank of an entry among equal codes of its
// wave comes from ballots on the code bits; waves are ordered through
// per-wave counts in LDS.  With mig_counts, also the segment's migration
// counts by direction code.  Called by the whole work-group (barriers
// inside); up to a work-group of leavers take two barriers.
template <typename R, int D, typename F>
__device__ __forceinline__ void bucket_outbox(const Params<R> &p, const int ts, const int n, F code_of,
                                              int *sBase, int *sCnt)
{
    // sBase: ncodes + 1 ints, sCnt: MAX_WAVES * ncodes ints of LDS
    constexpr int NC = ncodes<D>();
    constexpr int BITS = D == 1 ? 2 : (D == 2 ? 4 : 5);
    const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int32_t *boff = p.ob_boff + (int64_t)ts * (NC + 1);
    int32_t *idx = p.ob_idx + (int64_t)ts * p.ob_cap;
    for (int k = threadIdx.x; k < nw * NC; k += blockDim.x) sCnt[k] = 0;
    if (threadIdx.x < 64) {
        // bucket starts: a scan over the codes by the first wave
        const int c = threadIdx.x;
        const int v = c < NC ? sBase[c] : 0;
        int x = v;
#pragma unroll
        for (int o = 1; o < NC; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (c >= o) x += y;
        }
        if (c < NC) {
            sBase[c] = x - v;
            boff[c] = x - v;
            if (c == NC - 1) boff[NC] = x;
            // particles of the segment by the tile they went to: the outbox
            // buckets, and the stayers at the centre code (the segment count
            // before the arrivals are appended)
            if (p.mig_counts) p.mig_counts[(int64_t)ts * NC + c] = c == centre_code<D>() ? p.seg_cnt[ts] : v;
        }
    }
    __syncthreads();
    // stable scatter, one work-group-wide chunk at a time
    for (int c0 = 0; c0 < n; c0 += blockDim.x) {
        const int k = c0 + (int)threadIdx.x;
        const bool valid = k < n;
        const int code = valid ? code_of(k) : 0;
        unsigned long long m = __builtin_amdgcn_ballot_w64(valid);
#pragma unroll
        for (int b = 0; b < BITS; ++b) {
            const bool bit = (code >> b) & 1;
            const unsigned long long bb = __builtin_amdgcn_ballot_w64(bit);
            m &= bit ? bb : ~bb;
        }
        const int rank = lanes_below(m);
        if (valid && rank == 0) sCnt[wave * NC + code] = __popcll(m);
        __syncthreads();
        if (valid) {
            int off = sBase[code] + rank;
            for (int w = 0; w < wave; ++w) off += sCnt[w * NC + code];
            idx[off] = k;
        }
        if (c0 + (int)blockDim.x >= n) break;
        __syncthreads();
        if ((int)threadIdx.x < NC) {
            int add = 0;
            for (int w = 0; w < nw; ++w) {
                add += sCnt[w * NC + threadIdx.x];
                sCnt[w * NC + threadIdx.x] = 0;
            }
            sBase[threadIdx.x] += add;
        }
        __syncthreads();
    }
}

template <typename R, int D>
__device__ __forceinline__ bool inside_tile(const R x[3], const int32_t T[3])
{
    bool ok = true;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        R half = R(T[d] / 2);
        ok = ok && (x[d] >= -half) && (x[d] < half);   // false for NaN
    }
    return ok;
}

// A pushed particle may be deposited when each displacement is below one
// cell and the new position lies in the tile's current halo, so that the
// ZigZag stencil stays inside the LDS block (rounding of x + dx could
// otherwise reach the far face of the halo).
template <typename R, int D>
__device__ __forceinline__ bool moved_ok(const R x2[3], const R dv[3], const int32_t T[3])
{
    bool ok = true;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        R lim = R(T[d] / 2 + 1);
        ok = ok && fabs(dv[d]) < R(1) && x2[d] >= -lim && x2[d] < lim;
    }
    return ok;
}

template <typename R>
__device__ __forceinline__ bool finite3(const R v[3])
{
    return isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]);
}

// Write one chunk of particles after the push: stayers compacted in place
// (stable), leavers appended to the tile outbox rebased by -delta T.
// Must be called by every thread of the work-group.
template <typename R, int D>
__device__ __forceinline__ void compact_chunk(const Params<R> &p, int ts, int64_t so, bool valid, int code,
                                              const int delta[3], const R x2[3], const R u[3], int nvalid,
                                              int *sTot, int &parity, int &keep, int &nleave)
{
    const bool stay = valid && code == centre_code<D>();
    int tot;
    int pre = wg_scan_flag(stay, sTot, parity, tot);
    parity ^= 1;
    const int64_t cap = p.cap_total;
    if (stay) {
        int64_t dst = so + keep + pre;
#pragma unroll
        for (int d = 0; d < D; ++d) p.pos[d * cap + dst] = x2[d];
#pragma unroll
        for (int m = 0; m < 3; ++m) p.u[m * cap + dst] = u[m];
    } else if (valid) {
        int64_t slot = nleave + (threadIdx.x - pre);
        if (slot < p.ob_cap) {
            const int64_t ob = (int64_t)ts * p.ob_cap;
#pragma unroll
            for (int d = 0; d < D; ++d)
                p.ob_pos[(ob * D) + d * p.ob_cap + slot] = x2[d] - R(delta[d] * p.T[d]);
#pragma unroll
            for (int m = 0; m < 3; ++m) p.ob_u[(ob * 3) + m * p.ob_cap + slot] = u[m];
            p.ob_dir[(int64_t)ts * p.ob_dir_stride + slot] = code;
        } else {
            latch(p.err, ERR_CAPACITY);
        }
    }
    keep += tot;
    nleave += nvalid - tot;
}

// ------------------------------------------------------------------ push

// interp_em + push (+ comp_curr and particle pack when FUSED) for one tile.
// The current block is accumulated in LDS in type A: 64-bit fixed point for
// FP32 runs (exact integer adds, which gfx950's LDS also runs faster than
// its FP64 adds), FP64 for FP64 runs (the LDS FP32 atomic add is far slower
// than either under the many-address pattern of the deposit), or R on
// request; it is converted to R once, at the flush.  With HALFB the
// kernel applies push_half_b1 to its LDS copy of B itself (global B stays
// at B^{n-1/2}).  One particle per thread and group, the next group's loads
// in flight: two particles per thread, or a second group in flight, measured
// slower on the 2D FP32 push (the registers lower occupancy).
//
// Direction codes of the first p.dir_lds leavers stay in LDS (the bucketing
// at the end then reads nothing back from memory); the codes of later ones go
// to ob_dir.  DIR_LDS covers about twice the leavers of a segment of mean
// density (5% of 4,096 particles in a 16 x 16 tile, a fifth in an 8^3 tile).
template <int D>
__host__ __device__ constexpr int dir_lds()
{
    return D == 3 ? 2048 : 1024;
}

// LDS bytes of the push behind its field and current blocks, without the
// direction codes.
template <int D, bool FUSED>
__host__ __device__ constexpr int push_lds_tail()
{
    return (int)sizeof(int) * (2 * MAX_WAVES + 4 + (FUSED ? bucket_lds_ints<D>() : 0));
}

template <typename R, int D, bool FUSED, bool HALFB, typename A, int TC, bool WALLS, int PUSHER>
__device__ __forceinline__ void push_tile(const Params<R> &p, const int w, unsigned char *smem)
{
    constexpr int NC = ncodes<D>();
    // work item w = one (tile, species) segment
    const int t = w / p.nspecies, s = w - t * p.nspecies;
    if (!((p.species_mask >> s) & 1u)) return;   // species not pushed by this call
    const TileDesc td = p.tiles[t];
    // tile edge: a compile-time constant when TC > 0 (strides, LDS offsets
    // and the halves T/2 then fold into the instructions), else the runtime one
    int32_t T[3];
    if constexpr (TC > 0) {
        T[0] = TC;
        T[1] = D > 1 ? TC : 1;
        T[2] = D > 2 ? TC : 1;
    } else {
        T[0] = p.T[0];
        T[1] = p.T[1];
        T[2] = p.T[2];
    }
    const FieldBox<D> fb(T);
    const CurBox<D> cb(T);
    const bool planes = D == 3 || (TC == 0 && p.lds_planes);
    const FieldLds<D> fl(cb, fb, planes);
    const Strides js = cb.current();
    // the fields first: the immediate offsets of LDS read pairs (255 elements)
    // reach them only from a small base, those of the atomics reach 64 KB
    // (planes have an odd number of elements, so the current comes first)
    R *sF = reinterpret_cast<R *>(smem);
    A *sJ = reinterpret_cast<A *>(sF + 6 * cb.n);
    int *sTot = reinterpret_cast<int *>(sJ + (FUSED ? 3 * cb.n : 0));
    if (planes) {
        sJ = reinterpret_cast<A *>(smem);
        sF = reinterpret_cast<R *>(sJ + (FUSED ? 3 * cb.n : 0));
        sTot = reinterpret_cast<int *>(sF + 3 * cb.n + 3 * fb.n);
    }
    int *sNF = sTot + 2 * MAX_WAVES;             // particles left near a cell face
    int *sBase = sNF + 4;                        // leavers by direction code, then bucket starts
    int *sCnt = sBase + NC + 1;
    unsigned char *sDir = reinterpret_cast<unsigned char *>(sCnt + MAX_WAVES * NC);
    const int dir_cap = TC > 0 ? dir_lds<D>() : p.dir_lds;
    const int64_t cap = p.cap_total;
    const int G = blockDim.x, tid = threadIdx.x;
    // the segment's planes and its first group of particles.  Lanes past the
    // count read its last particle: loads need no branch.  FP32 loads the first group before the fields
    // are staged, so that both latencies overlap (measured: FP32 step 2 us
    // shorter; FP64 3-6 us longer, so FP64 loads them after the staging).
    const int64_t so = p.seg_off[w];
    const int cnt = p.seg_cnt[w];
    const R q = p.charge[td.box * p.nspecies + s];
    const R sq = p.qm[td.box * p.nspecies + s];
    // uniform base pointers of the segment's planes; particle slots are
    // 32-bit byte offsets from them (segment and outbox capacities are
    // bounded so that they fit)
    R *X[3], *V[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        X[d] = p.pos + (d < D ? d : 0) * cap + so;
        V[d] = p.u + d * cap + so;
    }
    constexpr bool EARLY = sizeof(R) == 4;
    R nx[3] = {0, 0, 0}, nu[3] = {0, 0, 0};
    auto load_group = [&](int c0, R *gx, R *gu) {
        const uint32_t o = (uint32_t)min(c0 + tid, cnt - 1) * (uint32_t)sizeof(R);
#pragma unroll
        for (int d = 0; d < D; ++d) gx[d] = ld_off(X[d], o);
#pragma unroll
        for (int m = 0; m < 3; ++m) gu[m] = ld_off(V[m], o);
    };
    if (EARLY && cnt > 0) load_group(0, nx, nu);
    stage_fields<R, D>(p.E, p.B, p.cells_total, td, T, sF, cb, fl);
    if (tid < 2 * MAX_WAVES) sTot[tid] = 0;
    if (tid == 0) *sNF = 0;
    if constexpr (FUSED) {
        for (int k = tid; k < 3 * cb.n; k += G) sJ[k] = A(0);
        if (tid < NC) sBase[tid] = 0;
    }
    __syncthreads();
    if constexpr (HALFB) {
        half_b_lds<R, D>(sF + fl.b0, fl.b, fb, sF, fl.e, R(0.5) * p.c, td, T, s == 0 ? p.bnext : nullptr,
                         p.cells_total);
        __syncthreads();
    }
    if constexpr (WALLS) {
        if (td.walls) {
            wall_images<R, D>(sF, cb, fb, fl, T, td.walls);
            __syncthreads();
        }
    }
    const R c = p.c, inv_c = p.inv_c;
    int parity = 0;
    int32_t errs = 0;
    int nfl = 0;         // this wave's particles left near a cell face
    int fx = 0;          // fixed-point exponent of the current block
    R qd = q;            // charge of the deposit: scaled by 2^e for a fixed-point block
    if constexpr (std::is_same<A, long long>::value) {
        fx = fixed_exponent(q);
        qd = ldexp(q, fx);
    }
    R *XO[3], *OX[3], *OU[3];
    const int64_t ob = (int64_t)w * p.ob_cap;
    const int ob_cap = (int)p.ob_cap;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        XO[d] = p.xold + (d < D ? d : 0) * cap + so;
        OX[d] = p.ob_pos + ob * D + (d < D ? d : 0) * p.ob_cap;
        OU[d] = p.ob_u + ob * 3 + d * p.ob_cap;
    }
    int32_t *const OD = p.ob_dir + (int64_t)w * p.ob_dir_stride;
    int keep = 0, nleave = 0;
    // The fused push writes a group's particles at the top of the next
    // iteration, before that iteration's prefetch.  The vector-memory
    // counter retires loads and stores in issue order, and a group's
    // stores depend on the lane masks (stayers, leavers): a wait for the
    // prefetched group would otherwise also wait for the stores issued just
    // before it.  Issued first, they complete under the next group's
    // compute.  (Stores go to compacted slots below the group just read,
    // and the prefetch reads beyond it.)
    struct Pending {
        bool stay, leave;
        uint32_t off;          // byte offset of the compacted or outbox slot
        R x[3], u[3];
    } pend;
    pend.stay = pend.leave = false;
    pend.off = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) pend.x[d] = pend.u[d] = R(0);
    auto flush_pending = [&](int c0) {   // c0: the pending group's first slot
        if (pend.stay) {
#pragma unroll
            for (int d = 0; d < D; ++d) st_off(X[d], pend.off, pend.x[d]);
#pragma unroll
            for (int m = 0; m < 3; ++m) st_off(V[m], pend.off, pend.u[m]);
            if (p.ids) st_off(p.ids + so, pend.off / (uint32_t)sizeof(R) * 4u, (int32_t)(so + c0 + tid));
        } else if (pend.leave) {
#pragma unroll
            for (int d = 0; d < D; ++d) st_off(OX[d], pend.off, pend.x[d]);
#pragma unroll
            for (int m = 0; m < 3; ++m) st_off(OU[m], pend.off, pend.u[m]);
            if (p.ids) st_off(p.ob_ids + ob, pend.off / (uint32_t)sizeof(R) * 4u, (int32_t)(so + c0 + tid));
        }
    };
    if (!EARLY && cnt > 0) load_group(0, nx, nu);
    int c0 = 0;
    for (; c0 < cnt; c0 += G) {
        const bool valid = c0 + tid < cnt;
        R x[3], u[3], xr[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            x[d] = nx[d];
            u[d] = nu[d];
        }
        if constexpr (FUSED) {
            // wait for this group's particles (and the stores issued with
            // them, a group ago) before issuing the previous group's
            // stores: s_waitcnt vmcnt(0), other counters untouched
            __builtin_amdgcn_s_waitcnt(0x0F70);
            flush_pending(c0 - G);
        }
        // prefetch: later groups lie beyond every element this group
        // writes (compaction only moves elements down)
        if (c0 + G < cnt) load_group(c0 + G, nx, nu);
        // end point in the tile's frame (unfused: not rebased), direction
        // code (-1 past the count); a particle with an error stays as it is
#pragma unroll
        for (int d = 0; d < 3; ++d) xr[d] = x[d];
        int code = -1;
        R face = R(1);       // distance to the nearest face beyond the near-face band
        if (valid) {
            code = centre_code<D>();
            bool ok = inside_tile<R, D>(x, T);
            if (!ok) errs |= ERR_OUT_OF_TILE;
            if (ok) {
                R e[3], b[3], dv[3], x2[3] = {x[0], x[1], x[2]};
                interp_all<R, D>(sF, fl, x, T, e, b);
                push_u<R, PUSHER>(u, e, b, c, inv_c, sq);
                R r;
                const R usq = displacement<R>(u, c, dv, r);
                end_point<R, D>(x, u, r, x2);
                // for finite momenta |dv_d| < c <= 1/sqrt(D), so the end point
                // stays in the current halo; 1 + |u|^2 is finite exactly when
                // u is.  Only a Courant number close to 1 (1D) can round a
                // displacement to a whole cell: then every move is checked.
                ok = isfinite(usq) && (c < R(0.99) || moved_ok<R, D>(x2, dv, T));
                if (!ok) errs |= isfinite(usq) ? ERR_CFL : ERR_NONFINITE;
                if (ok) {
                    if constexpr (FUSED) {
                        bool done = false;
                        if constexpr (WALLS) done = wall_reflect<R, D, A>(sJ, js, T, td.walls, x, x2, u, dv, qd);
                        if (!done) zigzag<R, D, A>(sJ, js, T, x, x2, dv, qd);
                        code = rebase<R, D>(x2, T, xr);
                    } else {
#pragma unroll
                        for (int d = 0; d < D; ++d) xr[d] = x2[d];
                    }
                }
            }
            // rebasing by -delta T (an even integer) is exact and keeps
            // the distance to the nearest face
            face = face_distance<R, D>(xr, p.nf_band);
        }
        nfl += __popcll(__builtin_amdgcn_ballot_w64(face <= R(0)));
        if constexpr (FUSED) {
            // stable compaction: stayers in place (every destination is at
            // or below an element this group has already read), leavers to
            // the outbox rebased by -delta T; written at the top of the next
            // iteration, under complementary lane masks (lanes past the
            // count write nothing)
            const bool stay = code == centre_code<D>();
            int tot;
            const int pre = wg_scan_flag(stay, sTot, parity, tot);
            parity ^= 1;
            pend.stay = stay;
            pend.leave = code >= 0 && !stay;
            int slot = stay ? keep + pre : nleave + (tid - pre);
            if (pend.leave) {
                if (slot < ob_cap) {
                    atomicAdd(&sBase[code], 1);
                    if (slot < dir_cap) sDir[slot] = (unsigned char)code;
                    else OD[slot] = code;
                } else {
                    errs |= ERR_CAPACITY;     // state is invalid from here on
                    slot = ob_cap - 1;
                }
            }
            pend.off = (uint32_t)slot * (uint32_t)sizeof(R);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                pend.x[d] = xr[d];
                pend.u[d] = u[d];
            }
            keep += tot;
            nleave += min(G, cnt - c0) - tot;
        } else if (valid) {
            const int i = c0 + tid;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                XO[d][i] = x[d];
                X[d][i] = xr[d];
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) V[m][i] = u[m];
        }
    }
    if constexpr (FUSED) flush_pending(c0 - G);            // the last group's stores
    latch_wave(p.err, errs);
    if ((tid & 63) == 0 && nfl) atomicAdd(sNF, nfl);
    // every wave's current, near-face counts and direction codes are complete
    __syncthreads();
    if (tid == 0) {
        p.nf_seg[w] = *sNF;
        if constexpr (FUSED) {
            p.seg_cnt[w] = keep;
            p.ob_cnt[w] = nleave;
        }
    }
    if constexpr (FUSED) {
        // the block goes out in its LDS layout, which the fold reads
        R *blk = p.jblk + (int64_t)w * 3 * cb.n;
        const double inv = std::is_same<A, long long>::value ? ldexp(1.0, -fx) : 1.0;
        for (int k = tid; k < 3 * cb.n; k += G) {
            if constexpr (std::is_same<A, long long>::value) blk[k] = (R)((double)sJ[k] * inv);
            else blk[k] = (R)sJ[k];
        }
        // bucket the outbox by direction code for the migration; codes beyond
        // the LDS list were stored by other waves of this group (the barrier
        // above makes them visible to it)
        bucket_outbox<R, D>(
            p, w, min(nleave, ob_cap), [&](int k) { return k < dir_cap ? (int)sDir[k] : OD[k]; }, sBase, sCnt);
    }
}

// Waves per SIMD the push is compiled for.  Two work-groups of 8^3 tiles fill
// the LDS; with 80 registers (walls need 89 unasked) they can hold 12 waves each.
template <typename R, int D, int TC>
__host__ __device__ constexpr int push_waves()
{
    return D == 3 && sizeof(R) == 4 && TC == 8 ? 6 : 4;
}

// One work-group per (tile, species) segment, segments dispatched in the
// order k_order wrote (largest particle count first).
// 1024^2 cells, 33.5 million particles, FP32: 390-397 us for 1.38 GB that it cannot
// do without (1.65 GB moved), bound by the particle stream and its compaction:
// without gathers and deposit it takes as long, without compaction 340 us, and a
// plain copy of the bytes 292 us.  8^3 tiles with walls, 29 million particles:
// 598 us (606 us with 512 threads and launches of their own for B and the arrivals), vector
// ALU 73% and LDS 69% busy.
template <typename R, int D, bool FUSED, bool HALFB, typename A, int TC, bool WALLS, int PUSHER>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(push_waves<R, D, TC>(), 8))) k_push(Params<R> p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    push_tile<R, D, FUSED, HALFB, A, TC, WALLS, PUSHER>(p, p.order[blockIdx.x], smem);
}

// Persistent walker: a grid sized to the resident work-groups pulls
// segments (largest first) from an atomic counter until every one is taken;
// every work-group leaves the loop when the counter passes the segment count.
// With walls it is compiled for 4 waves: the loop's own registers make it spill
// 17 at k_push's bound for 8^3 FP32 tiles (step of a 256x64x64 box of 8 particles
// per cell and species: 503 us, 474 us at 4 waves).  Without walls 2 spill there
// and the added waves are worth them (461 us, 467 us at 4 waves).
template <typename R, int D, bool FUSED, bool HALFB, typename A, int TC, bool WALLS, int PUSHER>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(WALLS ? 4 : push_waves<R, D, TC>(), 8)))
k_push_persistent(Params<R> p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int next;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(p.queue, 1);
        __syncthreads();
        const int k = next;
        __syncthreads();
        if (k >= p.ntiles * p.nspecies) break;
        push_tile<R, D, FUSED, HALFB, A, TC, WALLS, PUSHER>(p, p.order[k], smem);
        __syncthreads();
    }
}

// comp_curr after an unfused push: ZigZag from (xold, pos) of every
// particle into the segment's current block.  A lane takes four consecutive
// particles, one 16-byte load per plane (two at FP64), and the 16 lanes that
// the LDS serves together take quads 16 particles apart: particles sorted by
// cell otherwise send whole waves to one address (512^2, 16 particles per cell
// and species, sorted, FP32: 320 us with one particle per lane in order,
// 87 us now).  Two particles in 3D at FP64, where four need more than the 128
// registers of a 1,024-thread group (26 spilled; 64x48x40, 16 particles per cell
// and species, 4^3 tiles unsorted: 135 us with one particle per lane, 151 us with four,
// 101 us with two; 8^3 tiles sorted 305, 139 and 109 us).  In 1D and 2D FP64 four
// are better where particles are sorted (2D 8^2 tiles 70 us, 84 us with two).
template <typename R, int D, typename A>
__global__ void __launch_bounds__(1024) k_deposit(Params<R> p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int w = p.order[blockIdx.x];              // (tile, species) segment
    const int t = w / p.nspecies, s = w - t * p.nspecies;
    if (!((p.species_mask >> s) & 1u)) return;       // species not deposited by this call
    const TileDesc td = p.tiles[t];
    const CurBox<D> cb(p.T);
    A *sJ = reinterpret_cast<A *>(smem);
    for (int k = threadIdx.x; k < 3 * cb.n; k += blockDim.x) sJ[k] = A(0);
    __syncthreads();
    const int64_t cap = p.cap_total;
    const int64_t so = p.seg_off[w];
    const int cnt = p.seg_cnt[w];
    const R q = p.charge[td.box * p.nspecies + s];
    const int lane = threadIdx.x & 63;
    const int quad = ((lane & 15) << 2) | (lane >> 4);
    constexpr int NQ = D == 3 && sizeof(R) == 8 ? 2 : 4;
    // segments start at multiples of 64 slots and their capacities are
    // multiples of 64: every quad (or pair) of a count lies in its segment, aligned
    struct alignas(16) Quad {
        R v[NQ];
    };
    for (int i0 = ((threadIdx.x & ~63) + quad) * NQ; i0 < cnt; i0 += blockDim.x * NQ) {
        Quad a[D], b[D], u[3];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            a[d] = *reinterpret_cast<const Quad *>(p.xold + d * cap + so + i0);
            b[d] = *reinterpret_cast<const Quad *>(p.pos + d * cap + so + i0);
        }
#pragma unroll
        for (int m = 0; m < 3; ++m) u[m] = *reinterpret_cast<const Quad *>(p.u + m * cap + so + i0);
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            if (i0 + j >= cnt) break;
            R x1[3] = {0, 0, 0}, x2[3] = {0, 0, 0}, uu[3], dv[3], r;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                x1[d] = a[d].v[j];
                x2[d] = b[d].v[j];
            }
#pragma unroll
            for (int m = 0; m < 3; ++m) uu[m] = u[m].v[j];
            displacement<R>(uu, p.c, dv, r);
            const bool ok = inside_tile<R, D>(x1, p.T) && finite3<R>(uu) && moved_ok<R, D>(x2, dv, p.T);
            if (ok) zigzag<R, D, A>(sJ, cb.current(), p.T, x1, x2, dv, q);
        }
    }
    __syncthreads();
    R *blk = p.jblk + (int64_t)w * 3 * cb.n;
    for (int k = threadIdx.x; k < 3 * cb.n; k += blockDim.x) blk[k] = (R)sJ[k];
}

// Inputs of the E update at one cell: E there, B there (b) and B at the
// cell below along each axis a (bm[a]; the cell itself along axes at or
// beyond D), periodic inside the box.
template <typename R, int D>
__device__ __forceinline__ void load_e_update(const Params<R> &p, const R *B, const TileDesc &td, int gx, int gy,
                                              int gz, int64_t g, R e[3], R b[3], R bm[3][3])
{
    const int64_t N = p.cells_total;
    const int n0 = td.n[0], n1 = td.n[1], n2 = td.n[2];
    auto at = [&](int x, int y, int z) -> int64_t { return td.cell0 + x + (int64_t)n0 * (y + (int64_t)n1 * z); };
    const int64_t m[3] = {at(gx == 0 ? n0 - 1 : gx - 1, gy, gz), D > 1 ? at(gx, gy == 0 ? n1 - 1 : gy - 1, gz) : g,
                          D > 2 ? at(gx, gy, gz == 0 ? n2 - 1 : gz - 1) : g};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        e[c] = p.E[c * N + g];
        b[c] = B[c * N + g];
    }
    // the six neighbour values the curl uses
    bm[0][1] = B[N + m[0]];
    bm[0][2] = B[2 * N + m[0]];
    bm[1][0] = B[m[1]];
    bm[1][2] = B[2 * N + m[1]];
    bm[2][0] = B[m[2]];
    bm[2][1] = B[N + m[2]];
}

// E += h curl- B at one cell with the second-order backward differences of
// App. B, then E -= j when SUB_J; the tangential E vanishes on a wall plane.
// Takes the values load_e_update read.
template <typename R, int D, bool SUB_J>
__device__ __forceinline__ void update_e_cell(const Params<R> &p, const TileDesc &td, int gx, int64_t g, R h,
                                              const R j[3], const R e[3], const R b[3], const R bm[3][3])
{
    const int64_t N = p.cells_total;
    const R cx = (b[2] - bm[1][2]) - (b[1] - bm[2][1]);
    const R cy = (b[0] - bm[2][0]) - (b[2] - bm[0][2]);
    const R cz = (b[1] - bm[0][1]) - (b[0] - bm[1][0]);
    R ex = e[0] + h * cx, ey = e[1] + h * cy, ez = e[2] + h * cz;
    if constexpr (SUB_J) {
        ex -= j[0];
        ey -= j[1];
        ez -= j[2];
    }
    if ((td.walls & 1) && gx == 0) ey = ez = R(0);   // tangential E on the wall plane
    p.E[g] = ex;
    p.E[N + g] = ey;
    p.E[2 * N + g] = ez;
}

// E += h curl- B (- j) at one cell.
template <typename R, int D, bool SUB_J>
__device__ __forceinline__ void curl_b_update_e(const Params<R> &p, const TileDesc &td, int gx, int gy, int gz,
                                                int64_t g, R h, const R j[3])
{
    R e[3], b[3], bm[3][3];
    load_e_update<R, D>(p, p.B, td, gx, gy, gz, g, e, b, bm);
    update_e_cell<R, D, SUB_J>(p, td, gx, g, h, j, e, b, bm);
}

// B -= h curl+ E at one cell (global indices gx, gy, gz, storage index g),
// twice when TWICE (both half updates of Table 1 with the same E): the
// forward differences of App. B, periodic inside the box.  The new B goes to b.
template <typename R, int D, bool TWICE>
__device__ __forceinline__ void update_b_cell(const Params<R> &p, const TileDesc &td, int gx, int gy, int gz,
                                              int64_t g, R h, R b[3])
{
    const int64_t N = p.cells_total;
    const int n0 = td.n[0], n1 = td.n[1], n2 = td.n[2];
    auto at = [&](int x, int y, int z) -> int64_t { return td.cell0 + x + (int64_t)n0 * (y + (int64_t)n1 * z); };
    const R *Ex = p.E, *Ey = p.E + N, *Ez = p.E + 2 * N;
    const int64_t ip = D > 0 ? at(gx + 1 == n0 ? 0 : gx + 1, gy, gz) : g;
    const int64_t jp = D > 1 ? at(gx, gy + 1 == n1 ? 0 : gy + 1, gz) : g;
    const int64_t kp = D > 2 ? at(gx, gy, gz + 1 == n2 ? 0 : gz + 1) : g;
    const R ex = Ex[g], ey = Ey[g], ez = Ez[g];
    const R cx = (Ez[jp] - ez) - (Ey[kp] - ey);
    const R cy = (Ex[kp] - ex) - (Ez[ip] - ez);
    const R cz = (Ey[ip] - ey) - (Ex[jp] - ex);
    R bx = p.B[g], by = p.B[N + g], bz = p.B[2 * N + g];
    bx -= h * cx;
    by -= h * cy;
    bz -= h * cz;
    if constexpr (TWICE) {
        bx -= h * cx;
        by -= h * cy;
        bz -= h * cz;
    }
    b[0] = bx;
    b[1] = by;
    b[2] = bz;
}

// cur_exchange: J on the lattice = sum of the current blocks (one per
// species of species_mask) of the tile and of its neighbours whose halo covers the cell, in
// a fixed order (species, then neighbour offsets ascending, z major).  A
// block covers local cells -1..T+1, so along each dimension the tile below
// covers l < 2 and the tile above l = T-1.  The neighbours are walked one by
// one: a neighbour's block is the same for the whole work-group, so its
// address is scalar, a lane adds a 32-bit offset, and lanes (mostly whole
// waves) that the block does not cover skip the load.  One z layer of
// neighbours (9 blocks x 3 components) is in flight at a time.  With CURL_E the same pass
// also applies E += h curl- B - J to the cell (push_e and add_cur after the
// second half update of B), from the folded values still in registers: J
// is written once and not read back.
//
// NEXT_B: B after both half updates is read from p.bnext, where the push of
// a whole step left it, and the cell's own value is stored to B as well (no
// other work-group of the launch reads B).
template <typename R, int D, bool CURL_E, bool NEXT_B>
__device__ __forceinline__ void fold_tile(const Params<R> &p, R h, const int t)
{
    const TileDesc td = p.tiles[t];
    const CurBox<D> cb(p.T);
    const int T0 = p.T[0], T1 = D > 1 ? p.T[1] : 1, T2 = D > 2 ? p.T[2] : 1;
    const int ncell = T0 * T1 * T2;
    const float inv0 = 1.0f / T0, inv1 = 1.0f / T1;
    const Strides js = cb.current();
    const int64_t blk_len = 3 * (int64_t)cb.n;
    for (int k = threadIdx.x; k < ncell; k += blockDim.x) {
        const int r = D > 1 ? div_small(k, inv0) : 0, lz = D > 2 ? div_small(r, inv1) : 0;
        const int l[3] = {D > 1 ? k - r * T0 : k, D > 2 ? r - lz * T1 : r, lz};
        const int gx = td.tc[0] * T0 + l[0];
        const int gy = D > 1 ? td.tc[1] * T1 + l[1] : 0;
        const int gz = D > 2 ? td.tc[2] * T2 + l[2] : 0;
        const int64_t g = td.cell0 + gx + (int64_t)td.n[0] * (gy + (int64_t)td.n[1] * gz);
        // the E update's inputs first: loaded before the J stores below (which
        // the compiler may not move them across), all of the cell's loads are
        // in flight together
        R ee[3], eb[3], ebm[3][3];
        if constexpr (CURL_E) load_e_update<R, D>(p, NEXT_B ? p.bnext : p.B, td, gx, gy, gz, g, ee, eb, ebm);
        R acc[3] = {0, 0, 0};
        // the cell in its own tile's block, and per dimension whether the
        // tile below or above covers it
        const uint32_t own = (uint32_t)(l[0] + 1 + (D > 1 ? imul24(l[1] + 1, js.y) : 0) +
                                        (D > 2 ? imul24(l[2] + 1, js.z) : 0)) * (uint32_t)sizeof(R);
        bool cov[2][3];
#pragma unroll
        for (int d = 0; d < (D < 2 ? D : 2); ++d) {
            cov[d][0] = l[d] < 2;
            cov[d][1] = true;
            cov[d][2] = l[d] >= p.T[d] - 1;
        }
        for (int sp = 0; sp < p.nspecies; ++sp) {
            if (!((p.species_mask >> sp) & 1u)) continue;
#pragma unroll 1
            for (int oz = 0; oz < (D > 2 ? 3 : 1); ++oz) {
                constexpr int NY = D > 1 ? 3 : 1;
                const int wz = td.tc[2] + oz - 1;
                const int nz = D > 2 ? (wz < 0 ? wz + td.nt[2] : (wz >= td.nt[2] ? wz - td.nt[2] : wz)) : 0;
                if (D > 2 && !(oz == 0 ? l[2] < 2 : (oz == 1 || l[2] >= T2 - 1))) continue;
                R v[NY][3][3];
#pragma unroll
                for (int oy = 0; oy < NY; ++oy) {
                    const int wy = td.tc[1] + oy - 1;
                    const int ny = D > 1 ? (wy < 0 ? wy + td.nt[1] : (wy >= td.nt[1] ? wy - td.nt[1] : wy)) : 0;
#pragma unroll
                    for (int ox = 0; ox < 3; ++ox) {
                        const int wx = td.tc[0] + ox - 1;
                        const int nx = wx < 0 ? wx + td.nt[0] : (wx >= td.nt[0] ? wx - td.nt[0] : wx);
                        const int nid = td.tile0 + nx + td.nt[0] * (ny + td.nt[1] * nz);
                        // the neighbour's block, shifted so that the cell's
                        // entry lies at the same offset as in its own block
                        const int shift = (ox - 1) * T0 + (D > 1 ? (oy - 1) * T1 * js.y : 0) +
                                          (D > 2 ? (oz - 1) * T2 * js.z : 0);
                        const R *blk = p.jblk + (((int64_t)nid * p.nspecies + sp) * blk_len - shift);
#pragma unroll
                        for (int m = 0; m < 3; ++m) v[oy][ox][m] = R(0);
                        if (cov[0][ox] && (D < 2 || cov[1][oy])) {
#pragma unroll
                            for (int m = 0; m < 3; ++m) v[oy][ox][m] = ld_off(blk + m * js.m, own);
                        }
                    }
                }
#pragma unroll
                for (int oy = 0; oy < NY; ++oy)
#pragma unroll
                    for (int ox = 0; ox < 3; ++ox)
#pragma unroll
                        for (int m = 0; m < 3; ++m) acc[m] += v[oy][ox][m];
            }
        }
        p.J[g] = acc[0];
        p.J[p.cells_total + g] = acc[1];
        p.J[2 * p.cells_total + g] = acc[2];
        if constexpr (CURL_E) update_e_cell<R, D, true>(p, td, gx, g, h, acc, ee, eb, ebm);
        if constexpr (NEXT_B) {
#pragma unroll
            for (int m = 0; m < 3; ++m) p.B[m * p.cells_total + g] = eb[m];
        }
    }
}

template <typename R, int D, bool CURL_E>
__global__ void __launch_bounds__(256) k_fold(Params<R> p, R h)
{
    fold_tile<R, D, CURL_E, false>(p, h, xcd_tile(blockIdx.x, gridDim.x));
}

// ---------------------------------------------------------------- fields

// ORDER 2: the differences of App. B; ORDER 4: the fourth-order differences
// (FDTD4: weights 9/8 over one cell and -1/24 over three).
// PHASE 0: B -= h curl+ E.  PHASE 1: E += h curl- B.  PHASE 2: E -= J.
// PHASE 3: E += h curl- B - J.  PHASE 4: B -= h curl+ E twice (both half
// updates of Table 1 in one pass, same arithmetic as two PHASE 0 passes).
// (Eqs. fdB/fdE with the differences of App. B.)
template <typename R, int D, int PHASE, int ORDER>
__device__ __forceinline__ void field_tile(const Params<R> &p, R h, const int t)
{
    const TileDesc td = p.tiles[t];
    const int T0 = p.T[0], T1 = D > 1 ? p.T[1] : 1, T2 = D > 2 ? p.T[2] : 1;
    const int ncell = T0 * T1 * T2;
    const int64_t N = p.cells_total;
    const int n0 = td.n[0], n1 = td.n[1], n2 = td.n[2];
    for (int k = threadIdx.x; k < ncell; k += blockDim.x) {
        const int gx = td.tc[0] * T0 + k % T0;
        const int gy = D > 1 ? td.tc[1] * T1 + (k / T0) % T1 : 0;
        const int gz = D > 2 ? td.tc[2] * T2 + k / (T0 * T1) : 0;
        auto at = [&](int x, int y, int z) -> int64_t {
            return td.cell0 + x + (int64_t)n0 * (y + (int64_t)n1 * z);
        };
        const int64_t g = at(gx, gy, gz);
        // neighbour along axis a at offset o (periodic), and the differences
        auto nb = [&](int a, int o) -> int64_t {
            return a == 0 ? at(wrap_once(gx + o, n0), gy, gz) : a == 1 ? at(gx, wrap_once(gy + o, n1), gz) : at(gx, gy, wrap_once(gz + o, n2));
        };
        auto dfw = [&](const R *F, int a) -> R {
            if (a >= D) return R(0);
            if constexpr (ORDER == 4)
                return R(9.0 / 8.0) * (F[nb(a, 1)] - F[g]) - R(1.0 / 24.0) * (F[nb(a, 2)] - F[nb(a, -1)]);
            return F[nb(a, 1)] - F[g];
        };
        auto dbw = [&](const R *F, int a) -> R {
            if (a >= D) return R(0);
            if constexpr (ORDER == 4)
                return R(9.0 / 8.0) * (F[g] - F[nb(a, -1)]) - R(1.0 / 24.0) * (F[nb(a, 1)] - F[nb(a, -2)]);
            return F[g] - F[nb(a, -1)];
        };
        if constexpr (ORDER == 4 && (PHASE == 0 || PHASE == 4)) {
            const R *Ex = p.E, *Ey = p.E + N, *Ez = p.E + 2 * N;
            const R cx = dfw(Ez, 1) - dfw(Ey, 2), cy = dfw(Ex, 2) - dfw(Ez, 0), cz = dfw(Ey, 0) - dfw(Ex, 1);
            R bx = p.B[g] - h * cx, by = p.B[N + g] - h * cy, bz = p.B[2 * N + g] - h * cz;
            if constexpr (PHASE == 4) {
                bx -= h * cx;
                by -= h * cy;
                bz -= h * cz;
            }
            p.B[g] = bx;
            p.B[N + g] = by;
            p.B[2 * N + g] = bz;
        } else if constexpr (ORDER == 4 && (PHASE == 1 || PHASE == 3)) {
            const R *Bx = p.B, *By = p.B + N, *Bz = p.B + 2 * N;
            const R cx = dbw(Bz, 1) - dbw(By, 2), cy = dbw(Bx, 2) - dbw(Bz, 0), cz = dbw(By, 0) - dbw(Bx, 1);
            R ex = p.E[g] + h * cx, ey = p.E[N + g] + h * cy, ez = p.E[2 * N + g] + h * cz;
            if constexpr (PHASE == 3) {
                ex -= p.J[g];
                ey -= p.J[N + g];
                ez -= p.J[2 * N + g];
            }
            p.E[g] = ex;
            p.E[N + g] = ey;
            p.E[2 * N + g] = ez;
        } else if constexpr (PHASE == 0 || PHASE == 4) {
            R b[3];
            update_b_cell<R, D, PHASE == 4>(p, td, gx, gy, gz, g, h, b);
            p.B[g] = b[0];
            p.B[N + g] = b[1];
            p.B[2 * N + g] = b[2];
        } else if constexpr (PHASE == 2) {
            const bool wall = (td.walls & 1) && gx == 0;
            p.E[g] -= p.J[g];
            p.E[N + g] = wall ? R(0) : p.E[N + g] - p.J[N + g];
            p.E[2 * N + g] = wall ? R(0) : p.E[2 * N + g] - p.J[2 * N + g];
        } else {
            R j[3] = {0, 0, 0};
            if constexpr (PHASE == 3) {
                j[0] = p.J[g];
                j[1] = p.J[N + g];
                j[2] = p.J[2 * N + g];
            }
            curl_b_update_e<R, D, PHASE == 3>(p, td, gx, gy, gz, g, h, j);
        }
    }
}

template <typename R, int D, int PHASE, int ORDER = 2>
__global__ void __launch_bounds__(256) k_field(Params<R> p, R h)
{
    field_tile<R, D, PHASE, ORDER>(p, h, xcd_tile(blockIdx.x, gridDim.x));
}

// Fold of the current and, by the launch's second half of work-groups, the B
// update (PHASE 0 or 4) of a fused step: neither reads what the other writes.
template <typename R, int D, int PHASE, int ORDER>
__global__ void __launch_bounds__(256) k_fold_b(Params<R> p, R h)
{
    if ((int)blockIdx.x < p.ntiles) fold_tile<R, D, false, false>(p, R(0), xcd_tile(blockIdx.x, p.ntiles));
    else field_tile<R, D, PHASE, ORDER>(p, h, xcd_tile(blockIdx.x - p.ntiles, p.ntiles));
}

// Binomial current filter (the solver table's 3-point digital filter): one
// pass replaces every value by the (1/4, 1/2, 1/4) average along each grid
// dimension, i.e. the 3^D stencil of the product weights, periodic inside
// the box.  src and dst are [3][cells] planes and must differ.  One launch
// applies `passes` passes to a tile: it loads the tile with a halo of that many
// cells into LDS and lets the valid block shrink by a cell a pass (the same
// sums in the same order as pass by pass; the weights are powers of two).  A
// pass is far shorter than a launch: eight passes of 500x336 FP32 took 36 us as
// eight launches, 16 us as two of four.
template <typename R, int D>
__global__ void __launch_bounds__(256) k_filter(Params<R> p, const R *__restrict__ src, R *__restrict__ dst, int passes)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const TileDesc td = p.tiles[t];
    const int64_t N = p.cells_total;
    const int e0 = p.T[0] + 2 * passes, e1 = D > 1 ? p.T[1] + 2 * passes : 1, e2 = D > 2 ? p.T[2] + 2 * passes : 1;
    const int n = e0 * e1 * e2;
    const float inv0 = 1.0f / e0, inv1 = 1.0f / e1;
    R *a = reinterpret_cast<R *>(smem), *b = a + 3 * n;
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        int lx, ly, lz;
        cell_of<D>(k, e0, e1, inv0, inv1, lx, ly, lz);
        const int gx = wrap_near(td.tc[0] * p.T[0] + lx - passes, td.n[0]);
        const int gy = D > 1 ? wrap_near(td.tc[1] * p.T[1] + ly - passes, td.n[1]) : 0;
        const int gz = D > 2 ? wrap_near(td.tc[2] * p.T[2] + lz - passes, td.n[2]) : 0;
        const int64_t g = td.cell0 + gx + (int64_t)td.n[0] * (gy + (int64_t)td.n[1] * gz);
#pragma unroll
        for (int m = 0; m < 3; ++m) a[m * n + k] = src[m * N + g];
    }
    for (int q = 1; q <= passes; ++q) {
        __syncthreads();
        for (int k = threadIdx.x; k < n; k += blockDim.x) {
            int lx, ly, lz;
            cell_of<D>(k, e0, e1, inv0, inv1, lx, ly, lz);
            if (lx < q || lx >= e0 - q || (D > 1 && (ly < q || ly >= e1 - q)) || (D > 2 && (lz < q || lz >= e2 - q)))
                continue;
            R acc[3] = {0, 0, 0};
#pragma unroll
            for (int oz = (D > 2 ? -1 : 0); oz <= (D > 2 ? 1 : 0); ++oz)
#pragma unroll
                for (int oy = (D > 1 ? -1 : 0); oy <= (D > 1 ? 1 : 0); ++oy)
#pragma unroll
                    for (int ox = -1; ox <= 1; ++ox) {
                        const R w = (ox ? R(0.25) : R(0.5)) * (D > 1 ? (oy ? R(0.25) : R(0.5)) : R(1)) *
                                    (D > 2 ? (oz ? R(0.25) : R(0.5)) : R(1));
                        const int o = k + ox + e0 * (oy + e1 * oz);
#pragma unroll
                        for (int m = 0; m < 3; ++m) acc[m] += w * a[m * n + o];
                    }
            if (q < passes) {
#pragma unroll
                for (int m = 0; m < 3; ++m) b[m * n + k] = acc[m];
            } else {
                const int gx = td.tc[0] * p.T[0] + lx - passes;
                const int gy = D > 1 ? td.tc[1] * p.T[1] + ly - passes : 0;
                const int gz = D > 2 ? td.tc[2] * p.T[2] + lz - passes : 0;
                const int64_t g = td.cell0 + gx + (int64_t)td.n[0] * (gy + (int64_t)td.n[1] * gz);
#pragma unroll
                for (int m = 0; m < 3; ++m) dst[m * N + g] = acc[m];
            }
        }
        R *c = a;
        a = b;
        b = c;
    }
}

// One pass straight from memory, for tiles whose block does not fit the LDS.
template <typename R, int D>
__global__ void __launch_bounds__(256) k_filter_direct(Params<R> p, const R *__restrict__ src, R *__restrict__ dst)
{
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const TileDesc td = p.tiles[t];
    const int T0 = p.T[0], T1 = D > 1 ? p.T[1] : 1, T2 = D > 2 ? p.T[2] : 1;
    const int ncell = T0 * T1 * T2;
    const int64_t N = p.cells_total;
    const int n0 = td.n[0], n1 = td.n[1], n2 = td.n[2];
    for (int k = threadIdx.x; k < ncell; k += blockDim.x) {
        const int gx = td.tc[0] * T0 + k % T0;
        const int gy = D > 1 ? td.tc[1] * T1 + (k / T0) % T1 : 0;
        const int gz = D > 2 ? td.tc[2] * T2 + k / (T0 * T1) : 0;
        R acc[3] = {0, 0, 0};
        for (int oz = (D > 2 ? -1 : 0); oz <= (D > 2 ? 1 : 0); ++oz)
            for (int oy = (D > 1 ? -1 : 0); oy <= (D > 1 ? 1 : 0); ++oy)
                for (int ox = -1; ox <= 1; ++ox) {
                    const R w = (ox ? R(0.25) : R(0.5)) * (D > 1 ? (oy ? R(0.25) : R(0.5)) : R(1)) *
                                (D > 2 ? (oz ? R(0.25) : R(0.5)) : R(1));
                    const int64_t g = td.cell0 + wrap_once(gx + ox, n0) +
                                      (int64_t)n0 * (wrap_once(gy + oy, n1) + (int64_t)n1 * wrap_once(gz + oz, n2));
                    acc[0] += w * src[g];
                    acc[1] += w * src[N + g];
                    acc[2] += w * src[2 * N + g];
                }
        const int64_t g = td.cell0 + gx + (int64_t)n0 * (gy + (int64_t)n1 * gz);
        dst[g] = acc[0];
        dst[N + g] = acc[1];
        dst[2 * N + g] = acc[2];
    }
}

// ------------------------------------------------------------ migration

// Tag and pack outflowing particles after an unfused push (stable), one
// work-group per segment; a group's particles are loaded while the group
// before it is scanned and stored (stores go to slots below it).
template <typename R, int D>
__global__ void __launch_bounds__(1024) k_migrate_out(Params<R> p)
{
    __shared__ int sTot[2 * MAX_WAVES];
    const int ts = xcd_tile(blockIdx.x, gridDim.x);
    const int s = ts % p.nspecies;
    if (!((p.species_mask >> s) & 1u)) return;   // not pushed: every particle stayed
    const int64_t cap = p.cap_total;
    int parity = 0;
    if (threadIdx.x < 2 * MAX_WAVES) sTot[threadIdx.x] = 0;
    __syncthreads();
    const int64_t so = p.seg_off[ts];
    const int cnt = p.seg_cnt[ts];
    int keep = 0, nleave = 0;
    R nx[3] = {0, 0, 0}, nu[3] = {0, 0, 0};
    auto load = [&](int c0) {
        const int64_t i = so + min(c0 + (int)threadIdx.x, cnt - 1);
#pragma unroll
        for (int d = 0; d < D; ++d) nx[d] = p.pos[d * cap + i];
#pragma unroll
        for (int m = 0; m < 3; ++m) nu[m] = p.u[m * cap + i];
    };
    if (cnt > 0) load(0);
    for (int c0 = 0; c0 < cnt; c0 += blockDim.x) {
        const bool valid = c0 + (int)threadIdx.x < cnt;
        R x2[3], u[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            x2[d] = nx[d];
            u[d] = nu[d];
        }
        if (c0 + (int)blockDim.x < cnt) load(c0 + blockDim.x);
        int delta[3] = {0, 0, 0}, code = centre_code<D>();
        if (valid) code = direction_code<R, D>(x2, p.T, delta);
        const int nvalid = min((int)blockDim.x, cnt - c0);
        compact_chunk<R, D>(p, ts, so, valid, code, delta, x2, u, nvalid, sTot, parity, keep, nleave);
    }
    if (threadIdx.x == 0) {
        p.seg_cnt[ts] = keep;
        p.ob_cnt[ts] = nleave;
    }
}

// Bucket every segment's outbox by direction code (bucket_outbox), one
// work-group per segment, after an unfused push's k_migrate_out (the fused
// push buckets its own outbox at its end).
template <typename R, int D>
__global__ void __launch_bounds__(1024) k_migrate_bucket(Params<R> p)
{
    constexpr int NC = ncodes<D>();
    __shared__ int sScratch[bucket_lds_ints<D>()];
    int *sBase = sScratch, *sCnt = sBase + NC + 1;
    // one work-group per (tile, species) segment
    const int ts = xcd_tile(blockIdx.x, gridDim.x);
    // species_mask: the species pushed in this step; the outboxes of the
    // others hold nothing of this step
    const int s = ts % p.nspecies;
    const int n = ((p.species_mask >> s) & 1u) ? (int)min((int64_t)p.ob_cnt[ts], p.ob_cap) : 0;
    const int32_t *dir = p.ob_dir + (int64_t)ts * p.ob_dir_stride;
    if ((int)threadIdx.x < NC) sBase[threadIdx.x] = 0;
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += blockDim.x) atomicAdd(&sBase[dir[k]], 1);
    __syncthreads();
    bucket_outbox<R, D>(p, ts, n, [&](int k) { return dir[k]; }, sBase, sCnt);
}

// Migration counts by direction code after a fused push, from its bucket
// starts (before the arrivals are appended); species not pushed in the step
// count as staying.
template <typename R, int D>
__global__ void __launch_bounds__(256) k_migration_counts(Params<R> p)
{
    constexpr int NC = ncodes<D>();
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= (int64_t)p.ntiles * p.nspecies * NC) return;
    const int64_t ts = k / NC;
    const int c = (int)(k - ts * NC);
    const bool pushed = (p.species_mask >> (int)(ts % p.nspecies)) & 1u;
    const int32_t *boff = p.ob_boff + ts * (NC + 1);
    p.mig_counts[k] = c == centre_code<D>() ? p.seg_cnt[ts] : (pushed ? boff[c + 1] - boff[c] : 0);
}

// Receive incoming particles: append, per direction code in increasing
// order, the leavers of the neighbour that moved towards this tile (its
// bucket for that code, in the neighbour's order).  The buckets of all
// neighbours are walked as one index space (direction-major).
template <typename R, int D>
__device__ __forceinline__ void receive_segment(const Params<R> &p, const int ts)
{
    constexpr int NC = ncodes<D>();
    __shared__ int sOff[NC + 1];
    __shared__ int sSrc[NC];
    __shared__ int sB0[NC];
    const int t = ts / p.nspecies, s = ts - t * p.nspecies;
    const TileDesc td = p.tiles[t];
    const int64_t cap = p.cap_total;
    {
        const int64_t so = p.seg_off[ts];
        const int scap = p.seg_cap[ts];
        const int cnt = p.seg_cnt[ts];
        // the first wave: bucket sizes of the neighbours and their prefix
        // (a wave scan), one barrier
        if (threadIdx.x < 64) {
            const int code = threadIdx.x;
            int n_in = 0;
            if (code < NC) {
                int nc[3] = {0, 0, 0}, rem = code;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    if (d < D) {
                        const int delta = rem % 3 - 1;
                        rem /= 3;
                        const int v = td.tc[d] - delta;   // source tile, periodic (one step at most)
                        nc[d] = v < 0 ? v + td.nt[d] : (v >= td.nt[d] ? v - td.nt[d] : v);
                    }
                }
                const int sts = (td.tile0 + nc[0] + td.nt[0] * (nc[1] + td.nt[1] * nc[2])) * p.nspecies + s;
                const int32_t *boff = p.ob_boff + (int64_t)sts * (NC + 1);
                const int b0 = boff[code], b1 = boff[code + 1];   // both in flight before the LDS writes
                sSrc[code] = sts;
                sB0[code] = b0;
                // species not pushed in this step have no leavers (their
                // bucket starts may be an earlier step's)
                const bool pushed = (p.species_mask >> s) & 1u;
                n_in = code == centre_code<D>() || !pushed ? 0 : b1 - b0;
            }
            int x = n_in;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(x, o, 64);
                if (code >= o) x += y;
            }
            if (code < NC) sOff[code + 1] = x;
            if (code == 0) sOff[0] = 0;
        }
        __syncthreads();
        const int total = sOff[NC];
        int32_t errs = 0;
        for (int e = threadIdx.x; e < total; e += blockDim.x) {
            // code of element e: the first bucket whose end lies beyond e
            int code = 0, hi = NC - 1;
            while (code < hi) {
                const int mid = (code + hi) >> 1;
                if (sOff[mid + 1] <= e) code = mid + 1;
                else hi = mid;
            }
            const int64_t ob = (int64_t)sSrc[code] * p.ob_cap;
            const int64_t k = p.ob_idx[ob + sB0[code] + (e - sOff[code])];
            const int dst = cnt + e;
            if (dst < scap) {
                // every plane's load before the first store: the compiler
                // keeps a load behind an earlier store that it cannot tell
                // apart, and the planes then wait for one another
                R x[3], u[3];
                int32_t id = 0;
#pragma unroll
                for (int d = 0; d < D; ++d) x[d] = p.ob_pos[ob * D + d * p.ob_cap + k];
#pragma unroll
                for (int mm = 0; mm < 3; ++mm) u[mm] = p.ob_u[ob * 3 + mm * p.ob_cap + k];
                if (p.ids) id = p.ob_ids[ob + k];
#pragma unroll
                for (int d = 0; d < D; ++d) p.pos[d * cap + so + dst] = x[d];
#pragma unroll
                for (int mm = 0; mm < 3; ++mm) p.u[mm * cap + so + dst] = u[mm];
                if (p.ids) p.ids[so + dst] = id;
            } else {
                errs |= ERR_CAPACITY;
            }
        }
        if (errs) latch(p.err, errs);
        if (threadIdx.x == 0) p.seg_cnt[ts] = min(cnt + total, scap);
    }
}

// one work-group per (tile, species) segment
template <typename R, int D>
__global__ void __launch_bounds__(1024) k_migrate_in(Params<R> p)
{
    receive_segment<R, D>(p, xcd_tile(blockIdx.x, gridDim.x));
}

// Everything of a whole step after its fused push, in one launch: the first
// p.ntiles work-groups fold the current, advance E and store B (fold_tile),
// the others receive their segment's arrivals.  The two touch no common
// memory (blocks, E, B, J against outboxes and particles).
template <typename R, int D>
__global__ void __launch_bounds__(256) k_finish_step(Params<R> p, R h)
{
    if ((int)blockIdx.x < p.ntiles) fold_tile<R, D, true, true>(p, h, xcd_tile(blockIdx.x, p.ntiles));
    else receive_segment<R, D>(p, xcd_tile(blockIdx.x - p.ntiles, gridDim.x - p.ntiles));
}

// E update with the folded (and filtered) current, and the arrivals, likewise.
template <typename R, int D, int ORDER>
__global__ void __launch_bounds__(256) k_e_arrivals(Params<R> p, R h)
{
    if ((int)blockIdx.x < p.ntiles) field_tile<R, D, 3, ORDER>(p, h, xcd_tile(blockIdx.x, p.ntiles));
    else receive_segment<R, D>(p, xcd_tile(blockIdx.x - p.ntiles, gridDim.x - p.ntiles));
}

// Stable sort of every segment by cell index (x fastest), one work-group of up
// to SORT_WAVES waves per segment.  Each wave takes a contiguous share of the
// segment; per-wave cell histograms are scanned in (cell, wave) order, then
// each wave ranks its share in order, 64 particles at a time, equal keys among
// the lanes by ballots.  A segment of up to SORT_KEEP particles per thread
// keeps its keys and destinations in registers and is permuted plane by plane
// through an LDS buffer of buf elements: every plane is read and written once,
// coalesced, in place.  A larger one is scattered to the staging planes and
// copied back.  Bound by the planes' traffic (512^2, 16 particles per cell and
// species, FP32, 336 MB: 356 us with one group per tile, a serial scan and the
// staging planes for all, 97 us now).
constexpr int SORT_WAVES = 8;
constexpr int SORT_KEEP = 16;

template <typename R, int D>
__global__ void __launch_bounds__(64 * SORT_WAVES) k_cell_sort(Params<R> p, int buf)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int sWave[SORT_WAVES], sNF;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, nw = blockDim.x >> 6;
    const int T0 = p.T[0], T1 = D > 1 ? p.T[1] : 1, T2 = D > 2 ? p.T[2] : 1;
    const int ncell = T0 * T1 * T2;
    R *sV = reinterpret_cast<R *>(smem);
    int *hist = reinterpret_cast<int *>(sV + buf);      // [waves][ncell]
    int *mine = hist + wave * ncell;
    int nbits = 0;
    while ((1 << nbits) < ncell) ++nbits;
    const int64_t cap = p.cap_total;
    const int ts = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t so = p.seg_off[ts];
    const int cnt = p.seg_cnt[ts];
    const int per = (cnt + (int)blockDim.x - 1) / (int)blockDim.x * 64;   // of a wave
    const int lo = min(cnt, wave * per), hi = min(cnt, lo + per);
    const bool keep = per <= 64 * SORT_KEEP && cnt <= buf;
    if (tid == 0) sNF = 0;
    for (int k = tid; k < nw * ncell; k += blockDim.x) hist[k] = 0;
    __syncthreads();
    int nf = 0;
    auto key_of = [&](int i) -> int {
        R x[3] = {0, 0, 0};
        int key = 0, stride = 1;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            x[d] = p.pos[d * cap + so + i];
            const int c = min(max((int)floor(x[d]) + p.T[d] / 2, 0), p.T[d] - 1);
            key += c * stride;
            stride *= p.T[d];
        }
        nf += near_face<R, D>(x, p.nf_band);
        return key;
    };
    int key[SORT_KEEP];
    if (keep) {
#pragma unroll
        for (int j = 0; j < SORT_KEEP; ++j) {
            const int i = lo + j * 64 + lane;
            key[j] = -1;
            if (i < hi) key[j] = key_of(i);
        }
#pragma unroll
        for (int j = 0; j < SORT_KEEP; ++j)
            if (key[j] >= 0) atomicAdd(&mine[key[j]], 1);
    } else {
        for (int i = lo + lane; i < hi; i += 64) atomicAdd(&mine[key_of(i)], 1);
    }
    for (int o = 32; o > 0; o >>= 1) nf += __shfl_xor(nf, o);
    if (lane == 0 && nf) atomicAdd(&sNF, nf);
    __syncthreads();
    if (tid == 0) p.nf_seg[ts] = sNF;
    // exclusive scan in (cell, wave) order, a work-group of cells at a time
    int carry = 0;
    for (int c0 = 0; c0 < ncell; c0 += blockDim.x) {
        const int c = c0 + tid;
        int h[SORT_WAVES], tot = 0;
#pragma unroll
        for (int w = 0; w < SORT_WAVES; ++w) {
            h[w] = w < nw && c < ncell ? hist[w * ncell + c] : 0;
            tot += h[w];
        }
        int incl = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) sWave[wave] = incl;
        __syncthreads();
        int run = carry + incl - tot;
        for (int w = 0; w < nw; ++w) {
            run += w < wave ? sWave[w] : 0;
            carry += sWave[w];
        }
#pragma unroll
        for (int w = 0; w < SORT_WAVES; ++w) {
            if (w < nw && c < ncell) hist[w * ncell + c] = run;
            run += h[w];
        }
        __syncthreads();
    }
    // destination of a lane's particle: its cell's next slot for this wave
    // plus its rank among the equal keys of the 64
    auto rank_of = [&](int k) -> int {
        const bool valid = k >= 0;
        unsigned long long m = __builtin_amdgcn_ballot_w64(valid);
        for (int b = 0; b < nbits; ++b) {
            const bool bit = (k >> b) & 1;
            const unsigned long long bb = __builtin_amdgcn_ballot_w64(bit);
            m &= bit ? bb : ~bb;
        }
        int old = 0;
        if (valid) old = mine[k];
        const int below = lanes_below(m);
        if (valid && below == 0) mine[k] = old + __popcll(m);
        return old + below;
    };
    if (keep) {
        int dst[SORT_KEEP];
#pragma unroll
        for (int j = 0; j < SORT_KEEP; ++j) {
            dst[j] = -1;
            if (lo + j * 64 < hi) {                         // uniform in the wave
                const int r = rank_of(key[j]);
                if (key[j] >= 0) dst[j] = r;
            }
        }
#pragma unroll
        for (int pl = 0; pl < D + 3; ++pl) {
            R *P = pl < D ? p.pos + pl * cap + so : p.u + (pl - D) * cap + so;
            R v[SORT_KEEP];
#pragma unroll
            for (int j = 0; j < SORT_KEEP; ++j) {
                v[j] = R(0);
                if (dst[j] >= 0) v[j] = P[lo + j * 64 + lane];
            }
#pragma unroll
            for (int j = 0; j < SORT_KEEP; ++j)
                if (dst[j] >= 0) sV[dst[j]] = v[j];
            __syncthreads();
            for (int i = tid; i < cnt; i += blockDim.x) P[i] = sV[i];
            __syncthreads();
        }
        return;
    }
    for (int base = lo; base < hi; base += 64) {
        const int i = base + lane;
        const int r = rank_of(i < hi ? key_of(i) : -1);
        if (i < hi) {
            const int64_t dst = so + r;
#pragma unroll
            for (int d = 0; d < D; ++d) p.tmp[d * cap + dst] = p.pos[d * cap + so + i];
#pragma unroll
            for (int mm = 0; mm < 3; ++mm) p.tmp[(D + mm) * cap + dst] = p.u[mm * cap + so + i];
        }
    }
    __threadfence_block();
    __syncthreads();
    for (int i = tid; i < cnt; i += blockDim.x) {
        R v[D + 3];
#pragma unroll
        for (int d = 0; d < D + 3; ++d) v[d] = p.tmp[d * cap + so + i];
#pragma unroll
        for (int d = 0; d < D; ++d) p.pos[d * cap + so + i] = v[d];
#pragma unroll
        for (int mm = 0; mm < 3; ++mm) p.u[mm * cap + so + i] = v[D + mm];
    }
}

// Near-face count of every segment from its stored positions (after init,
// an injection, or before listing the flagged particles).
template <typename R, int D>
__global__ void __launch_bounds__(256) k_count_near_face(Params<R> p)
{
    __shared__ int sN;
    const int ts = blockIdx.x;
    const int64_t so = p.seg_off[ts];
    const int cnt = p.seg_cnt[ts];
    if (threadIdx.x == 0) sN = 0;
    __syncthreads();
    int nf = 0;
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
        R v[3] = {0, 0, 0};
#pragma unroll
        for (int d = 0; d < D; ++d) v[d] = p.pos[d * p.cap_total + so + i];
        nf += near_face<R, D>(v, p.nf_band);
    }
    for (int o = 32; o > 0; o >>= 1) nf += __shfl_xor(nf, o);
    if ((threadIdx.x & 63) == 0 && nf) atomicAdd(&sN, nf);
    __syncthreads();
    if (threadIdx.x == 0) p.nf_seg[ts] = sN;
}

// Exclusive prefix of the per-segment near-face counts (segment order, which
// is slot order) into pre, and the total into out[0].  One work-group.
__global__ void __launch_bounds__(1024) k_flag_scan(const int32_t *nf, int32_t n, int64_t *pre, int64_t *out)
{
    __shared__ int64_t wsum[16];
    __shared__ int64_t carry;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < n; base += 1024) {
        const int64_t v = base + tid < n ? nf[base + tid] : 0;
        int64_t x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wv] = x;
        __syncthreads();
        int64_t before = carry;
        for (int w = 0; w < wv; ++w) before += wsum[w];
        if (base + tid < n) pre[base + tid] = before + x - v;
        __syncthreads();
        if (tid == 0) {
            int64_t tot = 0;
            for (int w = 0; w < 16; ++w) tot += wsum[w];
            carry += tot;
        }
        __syncthreads();
    }
    if (tid == 0) out[0] = carry;
}

// Slots of the flagged particles, segment by segment in slot order, after
// k_flag_scan: flagged[1 + k] for k < capacity.  One work-group per segment;
// the order inside a segment comes from wave ballots and per-wave totals.
template <typename R, int D>
__global__ void __launch_bounds__(256) k_flag_list(Params<R> p, const int64_t *pre, int64_t *flagged, int64_t capacity)
{
    __shared__ int sTot[2 * MAX_WAVES];
    const int ts = blockIdx.x;
    const int64_t so = p.seg_off[ts];
    const int cnt = p.seg_cnt[ts];
    int64_t run = pre[ts];
    int parity = 0;
    if (threadIdx.x < 2 * MAX_WAVES) sTot[threadIdx.x] = 0;
    __syncthreads();
    for (int c0 = 0; c0 < cnt; c0 += blockDim.x) {
        const int i = c0 + threadIdx.x;
        bool f = false;
        if (i < cnt) {
            R v[3] = {0, 0, 0};
#pragma unroll
            for (int d = 0; d < D; ++d) v[d] = p.pos[d * p.cap_total + so + i];
            f = near_face<R, D>(v, p.nf_band);
        }
        int tot;
        const int k = wg_scan_flag(f, sTot, parity, tot);
        parity ^= 1;
        if (f && run + k < capacity) flagged[1 + run + k] = so + i;
        run += tot;
    }
}

}  // namespace pic
