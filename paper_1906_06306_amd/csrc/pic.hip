// libpic: C ABI of the MI355X relativistic PIC step (see include/pic.h).
//
// Host side: configuration checks, workspace layout, tile tables and kernel
// launches on the context's stream.  All device memory belongs to the
// caller's workspace; nothing here allocates device memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <limits>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/pic.h"
#include "pic_adjoint.hpp"
#include "pic_aux_kernels.hpp"

using pic::Params;
using pic::TileDesc;

namespace {

// largest segment or outbox capacity: the push addresses slots by 32-bit
// byte offsets from the segment's base, 8 * 2^28 bytes at FP64
constexpr int64_t MAX_SLOTS = int64_t(1) << 28;

// the segments' visiting order (largest first) only balances the push: any
// permutation gives the same results, and counts change by a few percent a
// step, so it is recomputed every ORDER_EVERY pushes, at the first push after
// init or an injection, and likewise inside a captured graph from its first push
// on (a replay of four steps on one stream, four boxes of 256 tiles in all, FP32:
// 179 us with an order at every captured push, 170 us)
constexpr int ORDER_EVERY = 8;

// text of the last error on this thread (a fixed buffer: reporting an
// error allocates nothing)
thread_local char g_last_error[512];

// Device scratch of pic_diagnostics_static, the diagnostics for callers that
// cannot allocate memory: the per-tile partial sums, the per-tile charge
// blocks and the reduced record.  Every device the library runs on holds
// one copy until the process ends; host code reaches a device's copy only
// through the address hipGetSymbolAddress returns for it (per device, at
// pic_init_tiles), never through the symbol itself.
constexpr uint64_t STATIC_SCRATCH_BYTES = uint64_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

std::mutex g_scratch_mu;
std::vector<void *> g_scratch_dev;   // device id -> address of that device's scratch

pic_status fail(pic_status code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof g_last_error, fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_OK(expr)                                                                          \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess) return fail(PIC_E_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

uint64_t align256(uint64_t v) { return (v + 255) & ~uint64_t(255); }

// Address of the current device's copy of `scratch` (looked up once per
// device, with that device current).
pic_status scratch_address(void **out)
{
    int dev = 0;
    HIP_OK(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if ((int)g_scratch_dev.size() <= dev) g_scratch_dev.resize(dev + 1, nullptr);
    if (!g_scratch_dev[dev]) {
        void *p = nullptr;
        HIP_OK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(PIC_E_HIP, "hipGetSymbolAddress returned a null address for the static scratch");
        g_scratch_dev[dev] = p;
    }
    *out = g_scratch_dev[dev];
    return PIC_OK;
}
int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// Internal layout: the public offsets plus the staging regions.
struct Layout {
    pic_layout pub;
    uint64_t off_tmp, off_jblk, off_rblk, off_part, off_ob_pos, off_ob_u, off_ob_dir, off_ob_cnt;
    uint64_t off_tiles, off_charge, off_qm, off_mass, off_order, off_queue;
    uint64_t off_key, off_xl, off_hist;
    uint64_t off_ob_ids, off_adj_lj, off_adj_eblk, off_adj_bblk, off_ob_boff, off_ob_idx, off_jtmp, off_rho_prev;
    uint64_t off_nf_pre;
    int64_t fblk_cells, n_input;
    int64_t jblk_cells, rblk_cells, max_count, max_ntb, nchunks_max, ob_dir_stride;
    int32_t order_shift;   // segment counts are bucketed by count >> order_shift for the dispatch order
    std::vector<TileDesc> tiles;
    std::vector<int64_t> seg_off;
    std::vector<int32_t> seg_cap;
    std::vector<int64_t> box_cell0, box_tile0;
    std::vector<int32_t> order;
};

int dims_of(const pic_config *c, int b, int d) { return d < c->dim ? c->box_cells[3 * b + d] : 1; }

pic_status check_config(const pic_config *c)
{
    if (!c) return fail(PIC_E_ARG, "null config");
    if (c->dim < 1 || c->dim > 3) return fail(PIC_E_ARG, "dim must be 1, 2 or 3 (got %d)", c->dim);
    if (c->precision != PIC_FP32 && c->precision != PIC_FP64) return fail(PIC_E_ARG, "precision must be PIC_FP32 or PIC_FP64");
    if (c->n_species < 1 || c->n_species > PIC_MAX_SPECIES) return fail(PIC_E_ARG, "n_species must be 1..%d", PIC_MAX_SPECIES);
    if (c->n_boxes < 1) return fail(PIC_E_ARG, "n_boxes must be >= 1");
    if (!c->box_cells || !c->charge || !c->qm || !c->mass) return fail(PIC_E_ARG, "box_cells, charge, qm and mass are required");
    if (!(c->cfl > 0.0) || c->cfl * std::sqrt((double)c->dim) > 1.0) return fail(PIC_E_ARG, "cfl must satisfy 0 < c <= 1/sqrt(D)");
    if (c->pusher < PIC_PUSHER_BORIS || c->pusher > PIC_PUSHER_HC) return fail(PIC_E_ARG, "unknown pusher %d", c->pusher);
    if (c->filter_passes < 0) return fail(PIC_E_ARG, "filter_passes must be >= 0");
    if (c->fdtd_order != 0 && c->fdtd_order != 2 && c->fdtd_order != 4) return fail(PIC_E_ARG, "fdtd_order must be 2 or 4");
    for (int b = 0; c->fdtd_order == 4 && c->box_walls && b < c->n_boxes; ++b)
        if (c->box_walls[b] & PIC_WALL_X) return fail(PIC_E_ARG, "FDTD4 covers periodic boxes only");
    for (int b = 0; c->filter_passes > 0 && c->box_walls && b < c->n_boxes; ++b)
        if (c->box_walls[b] & PIC_WALL_X) return fail(PIC_E_ARG, "the current filter covers periodic boxes only");
    int blk = c->block ? c->block : 256;
    if (blk < 64 || blk > 1024 || blk % 64) return fail(PIC_E_ARG, "block must be a multiple of 64 in 64..1024");
    for (int d = 0; d < 3; ++d) {
        if (d < c->dim) {
            if (c->tile[d] < 2 || c->tile[d] % 2) return fail(PIC_E_ARG, "tile[%d] must be even and >= 2", d);
        } else if (c->tile[d] != 1) {
            return fail(PIC_E_ARG, "tile[%d] must be 1 beyond dim", d);
        }
    }
    for (int b = 0; b < c->n_boxes; ++b)
        for (int d = 0; d < c->dim; ++d) {
            int n = c->box_cells[3 * b + d];
            if (n < c->tile[d] || n % c->tile[d]) return fail(PIC_E_ARG, "tile[%d]=%d does not divide box %d (n=%d)", d, c->tile[d], b, n);
        }
    return PIC_OK;
}

pic_status make_layout(const pic_config *c, const int64_t *counts, Layout &L)
{
    pic_status st = check_config(c);
    if (st) return st;
    if (!counts) return fail(PIC_E_ARG, "counts required");
    const int D = c->dim, ns = c->n_species, nb = c->n_boxes;
    const int64_t w = c->precision == PIC_FP64 ? 8 : 4;
    const int *T = c->tile;
    int64_t cells = 0, tiles = 0;
    L.box_cell0.assign(nb, 0);
    L.box_tile0.assign(nb, 0);
    L.tiles.clear();
    L.max_ntb = 0;
    L.max_count = 1;
    for (int b = 0; b < nb; ++b) {
        int n[3], nt[3];
        for (int d = 0; d < 3; ++d) {
            n[d] = dims_of(c, b, d);
            nt[d] = n[d] / T[d];
        }
        L.box_cell0[b] = cells;
        L.box_tile0[b] = tiles;
        int64_t ntb = (int64_t)nt[0] * nt[1] * nt[2];
        L.max_ntb = std::max(L.max_ntb, ntb);
        for (int tz = 0; tz < nt[2]; ++tz)
            for (int ty = 0; ty < nt[1]; ++ty)
                for (int tx = 0; tx < nt[0]; ++tx) {
                    TileDesc td{};
                    td.box = b;
                    td.tc[0] = tx, td.tc[1] = ty, td.tc[2] = tz;
                    for (int d = 0; d < 3; ++d) td.nt[d] = nt[d], td.n[d] = n[d];
                    td.cell0 = cells;
                    td.tile0 = (int32_t)tiles;
                    if (c->box_walls && (c->box_walls[b] & PIC_WALL_X))
                        td.walls = (tx == 0 ? 1 : 0) | (tx == nt[0] - 1 ? 2 : 0);
                    L.tiles.push_back(td);
                }
        cells += (int64_t)n[0] * n[1] * n[2];
        tiles += ntb;
        for (int s = 0; s < ns; ++s) {
            if (counts[b * ns + s] < 0) return fail(PIC_E_ARG, "negative particle count");
            L.max_count = std::max(L.max_count, counts[b * ns + s]);
            L.max_count = std::max<int64_t>(L.max_count, c->inject_max);
        }
    }
    if (L.max_ntb > (int64_t(1) << 24)) return fail(PIC_E_ARG, "a box has %lld tiles; at most 2^24 are supported", (long long)L.max_ntb);
    if (tiles > INT32_MAX / 8) return fail(PIC_E_ARG, "too many tiles");
    // segment capacities: a multiple of the block
    const int64_t group = c->block ? c->block : 256;
    double factor = c->capacity_factor > 0 ? c->capacity_factor : 1.25;
    L.seg_off.assign(tiles * ns, 0);
    L.seg_cap.assign(tiles * ns, 0);
    int64_t cap_total = 0, max_cap = 0;
    for (int64_t t = 0; t < tiles; ++t) {
        const int b = L.tiles[t].box;
        const int64_t ntb = (int64_t)L.tiles[t].nt[0] * L.tiles[t].nt[1] * L.tiles[t].nt[2];
        for (int s = 0; s < ns; ++s) {
            int64_t cap;
            if (c->tile_capacity) {
                cap = round_up(std::max<int64_t>(c->tile_capacity[t * ns + s], 64), group);
            } else {
                double expect = (double)counts[b * ns + s] / (double)ntb;
                cap = round_up((int64_t)std::ceil(factor * expect) + 64, group);
            }
            // the push addresses a segment's slots by 32-bit byte offsets
            if (cap > MAX_SLOTS) return fail(PIC_E_ARG, "segment capacity too large (at most 2^28 slots)");
            L.seg_off[t * ns + s] = cap_total;
            L.seg_cap[t * ns + s] = (int32_t)cap;
            cap_total += cap;
            max_cap = std::max(max_cap, cap);
        }
    }
    // segment visiting order before the first push (largest capacity first);
    // every push launch re-sorts the segments by their current counts
    L.order.resize(tiles * ns);
    for (int64_t w = 0; w < tiles * ns; ++w) L.order[w] = (int32_t)w;
    std::stable_sort(L.order.begin(), L.order.end(),
                     [&](int32_t a, int32_t b) { return L.seg_cap[a] > L.seg_cap[b]; });
    L.order_shift = 0;
    while ((max_cap >> L.order_shift) >= pic::ORDER_BUCKETS) ++L.order_shift;
    const int64_t obcap = c->outbox_capacity > 0 ? round_up(c->outbox_capacity, 64)
                                                 : round_up(std::max<int64_t>(256, max_cap / 4), 64);
    int64_t cb = 1, rb = 1;
    for (int d = 0; d < D; ++d) {
        cb *= T[d] + 3;
        rb *= T[d] + 1;
    }
    L.jblk_cells = cb;
    L.rblk_cells = rb;
    L.nchunks_max = std::min<int64_t>(2048, std::max<int64_t>(1, (L.max_count + 4095) / 4096));
    int64_t fbk = 1;
    for (int d = 0; d < D; ++d) fbk *= T[d] + 2;
    L.fblk_cells = fbk;
    L.n_input = 0;
    for (int i = 0; i < nb * ns; ++i) L.n_input += counts[i];
    const bool track = (c->options & PIC_OPT_TRACK) != 0;
    if (track && (cap_total > INT32_MAX || L.n_input > INT32_MAX))
        return fail(PIC_E_ARG, "origin tracking stores int32 ids: at most 2^31-1 slots and input particles");

    uint64_t off = 0;
    auto take = [&](uint64_t bytes) {
        uint64_t o = off;
        off = align256(off + std::max<uint64_t>(bytes, 1));
        return o;
    };
    pic_layout &P = L.pub;
    memset(&P, 0, sizeof P);
    P.off_E = take(3 * cells * w);
    P.off_B = take(3 * cells * w);
    P.off_J = take(3 * cells * w);
    P.off_pos = take(D * cap_total * w);
    P.off_u = take(3 * cap_total * w);
    P.off_xold = take(D * cap_total * w);
    P.off_seg_offset = take(tiles * ns * 8);
    P.off_seg_capacity = take(tiles * ns * 4);
    P.off_seg_count = take(tiles * ns * 4);
    P.off_error = take(4);
    P.off_flags = take(tiles * ns * 4);
    P.off_ids = take(track ? cap_total * 4 : 0);
    L.off_tmp = take((D + 3) * cap_total * w);
    L.off_jblk = take(tiles * ns * 3 * cb * w);
    L.off_rblk = take(tiles * rb * 8);
    L.off_part = take(tiles * pic::NPART * 8);
    L.off_ob_pos = take(tiles * ns * obcap * D * w);
    L.off_ob_u = take(tiles * ns * obcap * 3 * w);
    if (obcap > MAX_SLOTS) return fail(PIC_E_ARG, "outbox capacity too large (at most 2^28 slots)");
    L.ob_dir_stride = obcap;
    L.off_ob_dir = take(tiles * ns * L.ob_dir_stride * 4);
    L.off_ob_cnt = take(tiles * ns * 4);
    L.off_ob_boff = take(tiles * ns * (pic::ncodes<3>() + 1) * 4);
    L.off_ob_idx = take(tiles * ns * obcap * 4);
    L.off_jtmp = take(3 * cells * w);
    L.off_rho_prev = take(cells * 8);
    L.off_nf_pre = take(tiles * ns * 8);
    L.off_tiles = take(tiles * sizeof(TileDesc));
    L.off_charge = take(nb * ns * w);
    L.off_qm = take(nb * ns * w);
    L.off_mass = take(nb * ns * 8);
    L.off_order = take(tiles * ns * 4);
    L.off_queue = take(4);
    L.off_key = take(L.max_count * 4);
    L.off_xl = take(D * L.max_count * w);
    L.off_hist = take(L.nchunks_max * L.max_ntb * 4);
    L.off_ob_ids = take(track ? tiles * ns * obcap * 4 : 0);
    L.off_adj_lj = take(track ? 3 * cells * w : 0);
    L.off_adj_eblk = take(track ? tiles * 3 * cb * w : 0);
    L.off_adj_bblk = take(track ? tiles * 3 * fbk * w : 0);
    P.total_bytes = off;
    P.cells_total = cells;
    P.tiles_total = tiles;
    P.capacity_total = cap_total;
    P.outbox_capacity = obcap;
    P.elem_bytes = (int32_t)w;
    return PIC_OK;
}

}  // namespace

struct pic_ctx {
    int D, prec, ns, nb, block;
    bool acc_working;   // LDS current block in the working precision
    bool persistent;    // push as a persistent tile walker
    bool track;         // origin tracking and adjoint scratch present
    bool exact_block;   // the push takes block threads, not choose_group's
    bool walls;         // some box has conducting walls in x
    int pusher;         // PIC_PUSHER_*
    int filter_passes;  // binomial passes pic_step applies to J
    int order;          // FDTD order: 2 (App. B) or 4 (FDTD4)
    int64_t steps;      // completed steps
    int order_age;      // pushes since the visiting order was recomputed
    int64_t diag_step;  // steps at the last diagnostics call, or -1
    int n_cu;           // compute units of the device
    int push_group[2];  // threads per work-group of the unfused / fused push, 0 until its first launch
    hipGraphExec_t graph;   // captured steps, or null
    int graph_steps;
    int T[3];
    double c;
    Layout L;
    hipStream_t stream;
    uint8_t *ws;
    std::vector<double> mass;
    int state;          // 0 ready, 1 unfused push done, 2 fused push done, 3 unfused deposit done
    uint32_t all_species;   // mask of every species
    uint32_t pushed;        // species pushed in the current step
    uint32_t launch_mask;   // species of the next launch (Params::species_mask)
    bool step_b;            // the next push leaves B after both half updates in the scratch planes
    uint8_t *scratch;       // this device's static scratch (pic_diagnostics_static)
    double *pin;            // page-locked host memory for the diagnostic partials and, behind
                            // them, the error word: from the first call on, null where refused
};

namespace {

// Page-locked host memory, or null.  Another thread may be capturing a graph:
// the calls are no part of it.
void *page_locked(size_t bytes)
{
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    void *p = nullptr;
    if (hipHostMalloc(&p, bytes, hipHostMallocDefault) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    return p;
}

void free_page_locked(void *p)
{
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    (void)hipHostFree(p);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
}

template <typename R>
Params<R> params(pic_ctx *x)
{
    Params<R> p{};
    const Layout &L = x->L;
    uint8_t *ws = x->ws;
    p.tiles = reinterpret_cast<const TileDesc *>(ws + L.off_tiles);
    p.ntiles = (int32_t)L.pub.tiles_total;
    p.nspecies = x->ns;
    for (int d = 0; d < 3; ++d) p.T[d] = x->T[d];
    p.c = (R)x->c;
    p.inv_c = (R)(1.0 / x->c);
    p.charge = reinterpret_cast<const R *>(ws + L.off_charge);
    p.qm = reinterpret_cast<const R *>(ws + L.off_qm);
    p.E = reinterpret_cast<R *>(ws + L.pub.off_E);
    p.B = reinterpret_cast<R *>(ws + L.pub.off_B);
    p.J = reinterpret_cast<R *>(ws + L.pub.off_J);
    p.cells_total = L.pub.cells_total;
    p.pos = reinterpret_cast<R *>(ws + L.pub.off_pos);
    p.u = reinterpret_cast<R *>(ws + L.pub.off_u);
    p.xold = reinterpret_cast<R *>(ws + L.pub.off_xold);
    p.cap_total = L.pub.capacity_total;
    p.seg_off = reinterpret_cast<const int64_t *>(ws + L.pub.off_seg_offset);
    p.seg_cap = reinterpret_cast<const int32_t *>(ws + L.pub.off_seg_capacity);
    p.seg_cnt = reinterpret_cast<int32_t *>(ws + L.pub.off_seg_count);
    p.jblk = reinterpret_cast<R *>(ws + L.off_jblk);
    p.ob_pos = reinterpret_cast<R *>(ws + L.off_ob_pos);
    p.ob_u = reinterpret_cast<R *>(ws + L.off_ob_u);
    p.ob_dir = reinterpret_cast<int32_t *>(ws + L.off_ob_dir);
    p.ob_cnt = reinterpret_cast<int32_t *>(ws + L.off_ob_cnt);
    p.ob_boff = reinterpret_cast<int32_t *>(ws + L.off_ob_boff);
    p.ob_idx = reinterpret_cast<int32_t *>(ws + L.off_ob_idx);
    p.ob_cap = L.pub.outbox_capacity;
    p.ob_dir_stride = L.ob_dir_stride;
    p.tmp = reinterpret_cast<R *>(ws + L.off_tmp);
    p.err = reinterpret_cast<int32_t *>(ws + L.pub.off_error);
    p.nf_seg = reinterpret_cast<int32_t *>(ws + L.pub.off_flags);
    for (int d = 0; d < 3; ++d) {
        // 2 ulps of R at the tile half-width: every particle within 1 ulp of a
        // face, and every one that an FP32 step can move across a face
        // relative to the FP64 step from the same input
        const R h = (R)(x->T[d] / 2 > 0 ? x->T[d] / 2 : 1);
        p.nf_band[d] = R(2) * (std::nextafter(h, std::numeric_limits<R>::infinity()) - h);
    }
    p.species_mask = x->launch_mask;
    p.mig_counts = nullptr;
    p.queue = reinterpret_cast<int32_t *>(ws + L.off_queue);
    p.order = reinterpret_cast<int32_t *>(ws + L.off_order);
    if (x->track) {
        p.ids = reinterpret_cast<int32_t *>(ws + L.pub.off_ids);
        p.ob_ids = reinterpret_cast<int32_t *>(ws + L.off_ob_ids);
    }
    return p;
}

template <typename K>
pic_status set_lds(K kernel, size_t bytes)
{
    if (bytes > 160 * 1024) return fail(PIC_E_ARG, "tile needs %zu bytes of LDS (max 163840); use a smaller tile", bytes);
    if (bytes > 64 * 1024)
        HIP_OK(hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)bytes));
    return PIC_OK;
}

template <typename T>
pic_status fill(pic_ctx *x, T *p, int64_t n, T v)
{
    if (n <= 0) return PIC_OK;
    int grid = (int)std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(pic::k_fill<T>, dim3(grid), dim3(256), 0, x->stream, p, n, v);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

template <typename R, int D>
struct Impl {
    // LDS of the push (layout: push_tile), and for tiles with runtime edges the
    // choice of the layout: the first of interleaved rows with the direction
    // codes in LDS, the rows (planes in 3D) with the codes in memory, and one
    // plane per component, that leaves a CU as many work-groups as the last,
    // which is the smallest.  2D, 12 particles per cell and species: FP64 tiles of
    // 26x36, rows (one group) 655 us, planes (two) 610 us; FP32 of 38x38, rows with codes
    // 390 us, without (two) 343 us.
    template <int TC>
    static size_t push_lds(pic_ctx *x, Params<R> &p, bool fused, size_t acc_bytes)
    {
        int64_t fbn = 1, rows = 1, e0 = x->T[0] + 3;
        for (int d = 0; d < D; ++d) fbn *= x->T[d] + 2;
        for (int d = 1; d < D; ++d) rows *= x->T[d] + 3;
        const size_t tail = fused ? pic::push_lds_tail<D, true>() : pic::push_lds_tail<D, false>();
        const size_t cur = fused ? 3 * e0 * rows * acc_bytes : 0;
        const size_t planes = (3 * e0 * rows + 3 * fbn) * sizeof(R) + cur + tail;
        const size_t codes = fused ? pic::dir_lds<D>() : 0;
        const size_t lean = D == 3 ? planes : 6 * e0 * rows * sizeof(R) + cur + tail;
        // work-groups of the configured block that fit the LDS, which is handed
        // out in steps of 1,280 bytes, and the 32 waves of a CU
        auto groups = [&](size_t bytes) {
            return std::min<size_t>(160 * 1024 / ((bytes + 1279) / 1280 * 1280), 32 * 64 / x->block);
        };
        const size_t most = groups(planes);
        p.dir_lds = pic::dir_lds<D>();
        p.lds_planes = 0;
        if (TC > 0 || (most > 0 && groups(lean + codes) >= most)) return lean + codes;
        p.dir_lds = 0;
        if (most > 0 && groups(lean) >= most) return lean;
        p.lds_planes = 1;
        return planes;
    }

    template <int ORDER>
    static pic_status fdtd_order(pic_ctx *x, int phase)
    {
        Params<R> p = params<R>(x);
        dim3 g((unsigned)x->L.pub.tiles_total), b(256);
        const R c = (R)x->c;
        switch (phase) {
        case PIC_HALF_B: hipLaunchKernelGGL((pic::k_field<R, D, 0, ORDER>), g, b, 0, x->stream, p, R(0.5) * c); break;
        case PIC_CURL_E: hipLaunchKernelGGL((pic::k_field<R, D, 1, ORDER>), g, b, 0, x->stream, p, c); break;
        case PIC_ADD_J: hipLaunchKernelGGL((pic::k_field<R, D, 2, ORDER>), g, b, 0, x->stream, p, c); break;
        case PIC_CURL_E_ADD_J: hipLaunchKernelGGL((pic::k_field<R, D, 3, ORDER>), g, b, 0, x->stream, p, c); break;
        case PIC_TWO_HALF_B: hipLaunchKernelGGL((pic::k_field<R, D, 4, ORDER>), g, b, 0, x->stream, p, R(0.5) * c); break;
        default: return fail(PIC_E_ARG, "unknown fdtd phase %d", phase);
        }
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    static pic_status fdtd(pic_ctx *x, int phase)
    {
        return x->order == 4 ? fdtd_order<4>(x, phase) : fdtd_order<2>(x, phase);
    }

    // segments by decreasing count into p.order (one work-group)
    static pic_status order_segments(pic_ctx *x, const Params<R> &p)
    {
        hipLaunchKernelGGL(pic::k_order, dim3(1), dim3(pic::ORDER_BUCKETS), 0, x->stream, p.seg_cnt,
                           (int32_t)(x->L.pub.tiles_total * x->ns), x->L.order_shift, p.order);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // Threads per work-group of the push: the configured block, or more where that
    // puts more waves on a CU (the block doubled while below 256, then multiples
    // of 256 to 1,024; PIC_OPT_EXACT_BLOCK keeps the block).  A CU holds few groups
    // when the launch has few segments or LDS limits it; a larger group then fills
    // it (each group takes whole segments, so nothing else can).  Of equal
    // wave counts the larger group where the segments take at most two rounds of
    // resident groups (the largest segment ends the launch, and ends sooner), else
    // the smaller (fewer waves meet at the barrier of each group).  Step with the
    // block of 256 threads against the choice: 2D 256^2 FP32 (512 segments) 50.4 and
    // 46.9 us with 512; five steps and diagnostics of 512x384 (1,536 segments)
    // 615 and 606 us with 512; 3D FP64 box (480 segments, one group per CU)
    // 107.6 and 83.8 us with 1024; 512^2 FP64 with a block of 128 232 and 215 us
    // with 256.  1024^2 FP32 (8,192 segments) keeps 256: 512 takes 465 against
    // 451 us.  Where there are more rounds, only from half as many waves again: fewer
    // do not pay for the barriers and for the last, part-filled group of each
    // segment (3D FP64, 6^3 tiles of 1,080 particles, 128 registers: 996 us with 12
    // waves of 256 threads, 1,091 us with 16 of 512; of 2,160: 826 and 864 us; 2D 20x24
    // tiles alike, 604 and 600 us).
    // No larger than the particles a segment starts with (1D, 384 segments of 192
    // particles, FP32: push 7.7 us with 256 threads, 10.5 us with 1,024).  The host
    // knows only the counts at init: a run filled by injection keeps its block.
    // Three times 256 only where it fills a CU that the LDS leaves short of waves
    // (two groups of 8^3 FP32 tiles, 24 waves against 16: shock of 256x64x64 732
    // and 705 us); of few segments it would take room that other streams' launches
    // use (four boxes of 128^2 by graph replay on three streams: 103 us with 512,
    // 119 us with 768).
    template <typename K>
    static pic_status choose_group(pic_ctx *x, K kern, size_t lds, int64_t items, int &group)
    {
        if (group) return PIC_OK;
        if (x->exact_block) {
            group = x->block;
            return PIC_OK;
        }
        int best = x->block;
        int64_t best_waves = 0, block_waves = 0, most = 0;
        for (int g = x->block; g <= 1024; g = g < 256 ? 2 * g : (g / 256 + 1) * 256) {
            int per_cu = 0;
            HIP_OK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern), g, lds));
            const int64_t resident = std::max(per_cu, 1);
            const int64_t waves = std::min(resident, (items + x->n_cu - 1) / x->n_cu) * (g / 64);
            const bool two_rounds = items <= resident * x->n_cu * 2;
            const bool odd = (g & (g - 1)) && g != x->block && resident * (g / 64) <= most;
            most = std::max(most, resident * (g / 64));
            if (g > x->block && (int64_t)g * items > x->L.n_input) break;
            if (g == x->block) block_waves = waves;
            if (g > x->block && !two_rounds && 2 * waves < 3 * block_waves) continue;
            if (per_cu > 0 && !odd && (waves > best_waves || (waves == best_waves && two_rounds))) {
                best = g;
                best_waves = waves;
            }
        }
        group = best;
        return PIC_OK;
    }

    template <bool FUSED, bool HALFB, typename A, int TC, bool WALLS, int PUSHER>
    static pic_status push_launch(pic_ctx *x)
    {
        Params<R> p = params<R>(x);
        if (x->step_b) p.bnext = reinterpret_cast<R *>(x->ws + x->L.off_jtmp);
        size_t lds = push_lds<TC>(x, p, FUSED, sizeof(A));
        int &group = x->push_group[FUSED];
        const int64_t items = x->L.pub.tiles_total * x->ns;
        if (x->order_age >= ORDER_EVERY) {
            pic_status st0 = order_segments(x, p);
            if (st0) return st0;
            x->order_age = 0;
        }
        ++x->order_age;
        if (x->persistent) {
            auto kern = pic::k_push_persistent<R, D, FUSED, HALFB, A, TC, WALLS, PUSHER>;
            pic_status st = set_lds(kern, lds);
            if (st) return st;
            if ((st = choose_group(x, kern, lds, items, group))) return st;
            int per_cu = 0;
            HIP_OK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kern),
                                                                group, lds));
            const int64_t grid = std::min<int64_t>(items, (int64_t)std::max(per_cu, 1) * x->n_cu);
            st = fill<int32_t>(x, p.queue, 1, 0);
            if (st) return st;
            hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(group), lds, x->stream, p);
        } else {
            auto kern = pic::k_push<R, D, FUSED, HALFB, A, TC, WALLS, PUSHER>;
            pic_status st = set_lds(kern, lds);
            if (st || (st = choose_group(x, kern, lds, items, group))) return st;
            hipLaunchKernelGGL(kern, dim3((unsigned)items), dim3(group), lds, x->stream, p);
        }
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // The fused push with the 8-byte current block is compiled for the common cubic
    // tile edges with the edge as a constant; other shapes use the
    // runtime-edge kernel.
    template <bool FUSED, bool HALFB, typename A>
    static pic_status push_with(pic_ctx *x)
    {
        if (x->pusher == PIC_PUSHER_VAY)
            return x->walls ? push_launch<FUSED, HALFB, A, 0, FUSED, pic::PUSHER_VAY>(x)
                            : push_launch<FUSED, HALFB, A, 0, false, pic::PUSHER_VAY>(x);
        if (x->pusher == PIC_PUSHER_HC)
            return x->walls ? push_launch<FUSED, HALFB, A, 0, FUSED, pic::PUSHER_HC>(x)
                            : push_launch<FUSED, HALFB, A, 0, false, pic::PUSHER_HC>(x);
        bool cubic = true;
        for (int d = 1; d < D; ++d) cubic = cubic && x->T[d] == x->T[0];
        if constexpr (FUSED) {
            if (x->walls) {
                // the 3D shock's tiles: edge 8 as a constant
                if constexpr (D == 3 && (std::is_same<A, double>::value || std::is_same<A, long long>::value))
                    if (cubic && x->T[0] == 8) return push_launch<FUSED, HALFB, A, 8, true, pic::PUSHER_BORIS>(x);
                return push_launch<FUSED, HALFB, A, 0, true, pic::PUSHER_BORIS>(x);
            }
        }
        if constexpr (FUSED && (std::is_same<A, double>::value || std::is_same<A, long long>::value)) {
            if (cubic && x->T[0] == 8) return push_launch<FUSED, HALFB, A, 8, false, pic::PUSHER_BORIS>(x);
            if (cubic && x->T[0] == 16) return push_launch<FUSED, HALFB, A, 16, false, pic::PUSHER_BORIS>(x);
            if constexpr (D < 3)
                if (cubic && x->T[0] == 32) return push_launch<FUSED, HALFB, A, 32, false, pic::PUSHER_BORIS>(x);
        }
        return push_launch<FUSED, HALFB, A, 0, false, pic::PUSHER_BORIS>(x);
    }

    static pic_status push(pic_ctx *x, bool fused, bool halfb)
    {
        if (!fused) return halfb ? push_with<false, true, R>(x) : push_with<false, false, R>(x);
        if (x->acc_working) return halfb ? push_with<true, true, R>(x) : push_with<true, false, R>(x);
        // FP32: 64-bit fixed-point current block; FP64: FP64 block
        using Acc = typename std::conditional<sizeof(R) == 4, long long, double>::type;
        return halfb ? push_with<true, true, Acc>(x) : push_with<true, false, Acc>(x);
    }

    static pic_status deposit(pic_ctx *x, bool unfused_part, bool curl_e)
    {
        Params<R> p = params<R>(x);
        dim3 g((unsigned)x->L.pub.tiles_total);
        if (unfused_part) {
            const dim3 gs((unsigned)(x->L.pub.tiles_total * x->ns));   // one work-group per segment
            if (x->acc_working) {
                size_t lds = 3 * x->L.jblk_cells * sizeof(R);
                pic_status st = set_lds(pic::k_deposit<R, D, R>, lds);
                if (st) return st;
                hipLaunchKernelGGL((pic::k_deposit<R, D, R>), gs, dim3(x->block), lds, x->stream, p);
            } else {
                size_t lds = 3 * x->L.jblk_cells * sizeof(double);
                pic_status st = set_lds(pic::k_deposit<R, D, double>, lds);
                if (st) return st;
                hipLaunchKernelGGL((pic::k_deposit<R, D, double>), gs, dim3(x->block), lds, x->stream, p);
            }
            HIP_OK(hipGetLastError());
        }
        if (curl_e)
            hipLaunchKernelGGL((pic::k_fold<R, D, true>), g, dim3(256), 0, x->stream, p, (R)x->c);
        else
            hipLaunchKernelGGL((pic::k_fold<R, D, false>), g, dim3(256), 0, x->stream, p, R(0));
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // after the push of a whole step (step_b): fold, E update, B and arrivals
    static pic_status finish_step(pic_ctx *x)
    {
        Params<R> p = params<R>(x);
        p.bnext = reinterpret_cast<R *>(x->ws + x->L.off_jtmp);
        const dim3 g((unsigned)(x->L.pub.tiles_total * (1 + x->ns)));
        hipLaunchKernelGGL((pic::k_finish_step<R, D>), g, dim3(256), 0, x->stream, p, (R)x->c);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // The rest of a fused step with FDTD4 or the current filter, after the
    // push: fold with the B update, filter, E update with the arrivals (two
    // launches fewer than one by one: 500x336, eight passes, FDTD4, FP32
    // 79.5 and 72.8 us).  two_halves: B after both half updates (the push took the
    // first in LDS).
    template <int ORDER>
    static pic_status finish_rows_order(pic_ctx *x, bool two_halves)
    {
        Params<R> p = params<R>(x);
        const R c = (R)x->c;
        const dim3 g((unsigned)(2 * x->L.pub.tiles_total)), b(256);
        if (two_halves) hipLaunchKernelGGL((pic::k_fold_b<R, D, 4, ORDER>), g, b, 0, x->stream, p, R(0.5) * c);
        else hipLaunchKernelGGL((pic::k_fold_b<R, D, 0, ORDER>), g, b, 0, x->stream, p, R(0.5) * c);
        pic_status st = x->filter_passes ? filter(x, x->filter_passes) : PIC_OK;
        if (st) return st;
        const dim3 ga((unsigned)(x->L.pub.tiles_total * (1 + x->ns)));
        hipLaunchKernelGGL((pic::k_e_arrivals<R, D, ORDER>), ga, b, 0, x->stream, p, c);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    static pic_status finish_rows(pic_ctx *x, bool two_halves)
    {
        return x->order == 4 ? finish_rows_order<4>(x, two_halves) : finish_rows_order<2>(x, two_halves);
    }

    static pic_status migrate(pic_ctx *x, bool need_out, bool need_in, bool sort, int32_t *mig_counts,
                              int64_t *flagged, int64_t flagged_cap)
    {
        Params<R> p = params<R>(x);
        p.mig_counts = mig_counts;
        if (need_in) p.species_mask = x->pushed;   // only these species have leavers
        dim3 g((unsigned)x->L.pub.tiles_total);
        if (need_out) {
            // every group of particles ends in a scan: segments of many take
            // the largest work-group (512^2, 16 particles per cell and
            // species, FP32: 80 us with 256 threads, 70 with 512, 60)
            const int64_t segs = x->L.pub.tiles_total * x->ns;
            const int group = x->L.n_input >= segs * 1024 ? 1024 : x->block;
            hipLaunchKernelGGL((pic::k_migrate_out<R, D>), dim3((unsigned)segs), dim3(group), 0, x->stream, p);
            HIP_OK(hipGetLastError());
        }
        if (need_in) {
            // one small work-group per (tile, species) segment: both kernels
            // are chains of dependent loads, so many resident groups pay
            const dim3 gs((unsigned)(x->L.pub.tiles_total * x->ns));
            // the fused push buckets its own outbox; the unfused path runs the
            // bucket pass here (with the migration counts, if wanted)
            if (need_out)
                hipLaunchKernelGGL((pic::k_migrate_bucket<R, D>), gs, dim3(128), 0, x->stream, p);
            else if (mig_counts)
                hipLaunchKernelGGL((pic::k_migration_counts<R, D>),
                                   dim3((unsigned)((x->L.pub.tiles_total * x->ns * pic::ncodes<D>() + 255) / 256)),
                                   dim3(256), 0, x->stream, p);
            hipLaunchKernelGGL((pic::k_migrate_in<R, D>), gs, dim3(128), 0, x->stream, p);
            HIP_OK(hipGetLastError());
        }
        if (sort) {
            // per-wave cell histograms, and the permutation buffer: room for
            // SORT_KEEP particles per thread where the LDS has it (two
            // groups per CU); tiles of very many cells take half the waves
            const size_t cells = (size_t)x->T[0] * x->T[1] * x->T[2];
            const int waves = cells * pic::SORT_WAVES * sizeof(int) <= 64 * 1024 ? pic::SORT_WAVES : pic::SORT_WAVES / 2;
            const size_t hist = cells * waves * sizeof(int);
            int buf = 64 * waves * pic::SORT_KEEP;
            while (buf > 0 && hist + buf * sizeof(R) > 80 * 1024) buf /= 2;
            const size_t lds = hist + buf * sizeof(R);
            pic_status st = set_lds(pic::k_cell_sort<R, D>, lds);
            if (st) return st;
            hipLaunchKernelGGL((pic::k_cell_sort<R, D>), dim3((unsigned)(x->L.pub.tiles_total * x->ns)),
                               dim3(64 * waves), lds, x->stream, p, buf);
            HIP_OK(hipGetLastError());
        }
        if (flagged) {
            // per-segment counts of the stored positions, their prefix in
            // slot order (and the total into flagged[0]), then the slots
            const int64_t nseg = x->L.pub.tiles_total * x->ns;
            int64_t *pre = reinterpret_cast<int64_t *>(x->ws + x->L.off_nf_pre);
            hipLaunchKernelGGL((pic::k_count_near_face<R, D>), dim3((unsigned)nseg), dim3(256), 0, x->stream, p);
            hipLaunchKernelGGL(pic::k_flag_scan, dim3(1), dim3(1024), 0, x->stream, p.nf_seg, (int32_t)nseg, pre,
                               flagged);
            hipLaunchKernelGGL((pic::k_flag_list<R, D>), dim3((unsigned)nseg), dim3(256), 0, x->stream, p, pre,
                               flagged, flagged_cap);
            HIP_OK(hipGetLastError());
        }
        return PIC_OK;
    }

    // near-face count of every segment from the stored positions
    static pic_status count_near_face(pic_ctx *x)
    {
        Params<R> p = params<R>(x);
        hipLaunchKernelGGL((pic::k_count_near_face<R, D>), dim3((unsigned)(x->L.pub.tiles_total * x->ns)), dim3(256),
                           0, x->stream, p);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // Bin count FP64 particles of (box b, species s) into their tiles and
    // append them to the segments (after the particles already there, input
    // order kept inside a tile); origin ids id_base + i, or -1 if id_base < 0.
    static pic_status bin_species(pic_ctx *x, int b, int s, int64_t count, const double *pos, const double *u,
                                  int64_t id_base)
    {
        Params<R> p = params<R>(x);
        const Layout &L = x->L;
        uint8_t *ws = x->ws;
        int32_t *key = reinterpret_cast<int32_t *>(ws + L.off_key);
        R *xl = reinterpret_cast<R *>(ws + L.off_xl);
        int32_t *hist = reinterpret_cast<int32_t *>(ws + L.off_hist);
        const TileDesc &t0 = L.tiles[L.box_tile0[b]];
        pic::BinGeom g{};
        for (int d = 0; d < 3; ++d) {
            g.n[d] = t0.n[d];
            g.T[d] = x->T[d];
            g.nt[d] = t0.nt[d];
        }
        g.ntb = t0.nt[0] * t0.nt[1] * t0.nt[2];
        g.count = count;
        g.nchunks = (int32_t)std::min<int64_t>(L.nchunks_max, std::max<int64_t>(1, (count + 4095) / 4096));
        g.chunk = (int32_t)((count + g.nchunks - 1) / g.nchunks);
        g.id_base = id_base;
        g.walls = L.tiles[L.box_tile0[b]].walls != 0 || L.tiles[L.box_tile0[b] + t0.nt[0] - 1].walls != 0;
        int kgrid = (int)std::min<int64_t>((count + 255) / 256, 16384);
        hipLaunchKernelGGL((pic::k_bin_keys<R, D>), dim3(kgrid), dim3(256), 0, x->stream, g, pos, key, xl, p.err);
        // per-chunk tile histograms in LDS up to 32,768 tiles per box, else
        // in global memory (zeroed here)
        g.hist_lds = g.ntb <= 32768;
        size_t lds = g.hist_lds ? (size_t)g.ntb * sizeof(int) : 0;
        pic_status st = PIC_OK;
        if (!g.hist_lds) st = fill<int32_t>(x, hist, (int64_t)g.nchunks * g.ntb, 0);
        if (!st) st = set_lds(pic::k_bin_hist, lds);
        if (st) return st;
        hipLaunchKernelGGL(pic::k_bin_hist, dim3(g.nchunks), dim3(256), lds, x->stream, g, key, hist);
        hipLaunchKernelGGL(pic::k_bin_scan, dim3((g.ntb + 63) / 64), dim3(64), 0, x->stream, g, hist, p.seg_cnt,
                           p.seg_cap, (int)L.box_tile0[b], x->ns, s, p.err);
        st = set_lds(pic::k_bin_scatter<R, D>, lds);
        if (st) return st;
        hipLaunchKernelGGL((pic::k_bin_scatter<R, D>), dim3(g.nchunks), dim3(64), lds, x->stream, g, key, xl, u, hist, p,
                           (int)L.box_tile0[b], s);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    static pic_status inject(pic_ctx *x, int b, int s, int64_t count, const double *pos, const double *u)
    {
        pic_status st = bin_species(x, b, s, count, pos, u, -1);
        return st ? st : count_near_face(x);
    }

    static pic_status init(pic_ctx *x, const int64_t *counts, const pic_init_data *in)
    {
        Params<R> p = params<R>(x);
        const Layout &L = x->L;
        pic_status st = fill<int32_t>(x, p.seg_cnt, L.pub.tiles_total * x->ns, 0);
        if (!st) st = fill<int32_t>(x, p.ob_cnt, L.pub.tiles_total * x->ns, 0);
        if (!st) st = fill<R>(x, p.J, 3 * L.pub.cells_total, R(0));
        if (!st) st = fill<R>(x, p.E, 3 * L.pub.cells_total, R(0));
        if (!st) st = fill<R>(x, p.B, 3 * L.pub.cells_total, R(0));
        if (!st) st = fill<R>(x, p.jblk, L.pub.tiles_total * x->ns * 3 * L.jblk_cells, R(0));
        if (st) return st;
        int64_t id_base = 0;
        for (int b = 0; b < x->nb; ++b) {
            const TileDesc &t0 = L.tiles[L.box_tile0[b]];
            const int64_t cells = (int64_t)t0.n[0] * t0.n[1] * t0.n[2];
            int grid = (int)std::min<int64_t>((3 * cells + 255) / 256, 8192);
            if (in->E && in->E[b])
                hipLaunchKernelGGL((pic::k_load_field<R>), dim3(grid), dim3(256), 0, x->stream, p.E, L.pub.cells_total,
                                   L.box_cell0[b], in->E[b], cells);
            if (in->B && in->B[b])
                hipLaunchKernelGGL((pic::k_load_field<R>), dim3(grid), dim3(256), 0, x->stream, p.B, L.pub.cells_total,
                                   L.box_cell0[b], in->B[b], cells);
            HIP_OK(hipGetLastError());
            for (int s = 0; s < x->ns; ++s) {
                const int64_t count = counts[b * x->ns + s];
                id_base += count;
                if (count == 0) continue;
                if (!in->pos || !in->u || !in->pos[b * x->ns + s] || !in->u[b * x->ns + s])
                    return fail(PIC_E_ARG, "missing particle data for box %d species %d", b, s);
                st = bin_species(x, b, s, count, in->pos[b * x->ns + s], in->u[b * x->ns + s], id_base - count);
                if (st) return st;
            }
        }
        if (x->walls) {
            hipLaunchKernelGGL((pic::k_hold_walls<R, D>), dim3((unsigned)L.pub.tiles_total), dim3(256), 0, x->stream, p);
            HIP_OK(hipGetLastError());
        }
        return count_near_face(x);
    }

    // offsets of a state image (pic_state_save): E, B, pos, u, counts, error,
    // near-face counts, ids
    static uint64_t image_offsets(pic_ctx *x, uint64_t off[8])
    {
        const pic_layout &P = x->L.pub;
        const uint64_t nseg = P.tiles_total * x->ns;
        const uint64_t bytes[8] = {3 * P.cells_total * sizeof(R),  3 * P.cells_total * sizeof(R),
                                   D * P.capacity_total * sizeof(R), 3 * P.capacity_total * sizeof(R),
                                   nseg * sizeof(int32_t), sizeof(int32_t), nseg * sizeof(int32_t),
                                   P.capacity_total * sizeof(int32_t)};
        uint64_t o = 0;
        for (int k = 0; k < 8; ++k) {
            off[k] = o;
            o = align256(o + bytes[k]);
        }
        return o;
    }

    static pic_status state_bytes(pic_ctx *x, uint64_t *out)
    {
        uint64_t off[8];
        *out = image_offsets(x, off);
        return PIC_OK;
    }

    static pic::StateView<R> image_view(pic_ctx *x, const void *image)
    {
        uint64_t o[8];
        image_offsets(x, o);
        uint8_t *b = static_cast<uint8_t *>(const_cast<void *>(image));
        return {reinterpret_cast<R *>(b + o[0]), reinterpret_cast<R *>(b + o[1]), reinterpret_cast<R *>(b + o[2]),
                reinterpret_cast<R *>(b + o[3]), reinterpret_cast<int32_t *>(b + o[4]),
                reinterpret_cast<int32_t *>(b + o[5]), reinterpret_cast<int32_t *>(b + o[6]),
                reinterpret_cast<int32_t *>(b + o[7])};
    }

    static pic_status state_copy(pic_ctx *x, void *image, bool save)
    {
        const Params<R> p = params<R>(x);
        const pic::StateView<R> ws = {p.E, p.B, p.pos, p.u, p.seg_cnt, p.err, p.nf_seg, p.ids}, im = image_view(x, image);
        const int32_t nseg = (int32_t)(x->L.pub.tiles_total * x->ns);
        const int64_t cells = x->L.pub.cells_total;
        const unsigned nf = (unsigned)std::min<int64_t>(std::max<int64_t>(1, (3 * cells + 1023) / 1024), 2048);
        hipLaunchKernelGGL((pic::k_state_copy<R, D>), dim3((unsigned)nseg + nf), dim3(256), 0, x->stream,
                           save ? im : ws, save ? ws : im, p.seg_off, nseg, x->L.pub.capacity_total, cells,
                           save ? 0 : 1);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // Reverse of one fused step from the current state (Table 1 rows in
    // reverse order; the field rows reuse the forward stencils on the
    // adjoint fields, since (curl+)^T = curl- on the periodic lattice).
    // With an image the state is read there; with opos and ou the particle
    // adjoints go to the slots the particles came from.
    template <int TC>
    static pic_status adj_push(pic_ctx *x, const Params<R> &p, const pic::AdjParams<R> &a, size_t lds)
    {
        pic_status st = set_lds(pic::k_adj_push<R, D, TC>, lds);
        if (st) return st;
        hipLaunchKernelGGL((pic::k_adj_push<R, D, TC>), dim3((unsigned)x->L.pub.tiles_total),
                           dim3(pic::adj_block<R, D>()), lds, x->stream, p, a);
        return PIC_OK;
    }

    static pic_status adjoint(pic_ctx *x, void *lpos, void *lu, void *lE, void *lB, const void *image, void *opos,
                              void *ou, int64_t ostride)
    {
        Params<R> p = params<R>(x);
        if (image) {
            const pic::StateView<R> v = image_view(x, image);
            p.E = v.E;
            p.B = v.B;
            p.pos = v.pos;
            p.u = v.u;
            p.seg_cnt = v.seg_cnt;
            p.ids = v.ids;
        }
        const Layout &L = x->L;
        pic::AdjParams<R> a{};
        a.opos = reinterpret_cast<R *>(opos);
        a.ou = reinterpret_cast<R *>(ou);
        a.ostride = ostride;
        a.lpos = reinterpret_cast<R *>(lpos);
        a.lu = reinterpret_cast<R *>(lu);
        a.lE = reinterpret_cast<R *>(lE);
        a.lB = reinterpret_cast<R *>(lB);
        a.lJ = reinterpret_cast<R *>(x->ws + L.off_adj_lj);
        a.eblk = reinterpret_cast<R *>(x->ws + L.off_adj_eblk);
        a.bblk = reinterpret_cast<R *>(x->ws + L.off_adj_bblk);
        dim3 g((unsigned)L.pub.tiles_total), b(256);
        // comp_curr, position update, Boris, interp_em per particle
        const size_t lds = 3 * (L.jblk_cells + L.fblk_cells) * sizeof(double) +
                           (6 * L.jblk_cells + 3 * L.fblk_cells) * sizeof(R);
        bool cubic = true;
        for (int d = 1; d < D; ++d) cubic = cubic && x->T[d] == x->T[0];
        const int edge = cubic ? x->T[0] : 0;
        pic_status st = edge == 8 ? adj_push<8>(x, p, a, lds) : edge == 16 ? adj_push<16>(x, p, a, lds) : adj_push<0>(x, p, a, lds);
        if (st) return st;
        hipLaunchKernelGGL((pic::k_adj_fields<R, D, true>), g, b, 0, x->stream, p, a);
        hipLaunchKernelGGL((pic::k_adj_fields<R, D, false>), g, b, 0, x->stream, p, a);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    static size_t filter_lds(pic_ctx *x, int passes)
    {
        size_t n = 1;
        for (int d = 0; d < D; ++d) n *= x->T[d] + 2 * passes;
        return 2 * 3 * n * sizeof(R);
    }

    // The passes in an even number of launches (each reads one of J and the
    // scratch planes and writes the other), up to MOST passes a launch: the
    // halo's share of the work grows with them, and in 3D with its cube.
    static pic_status filter(pic_ctx *x, int passes)
    {
        constexpr int MOST = D == 1 ? 8 : (D == 2 ? 4 : 2);
        Params<R> p = params<R>(x);
        R *tmp = reinterpret_cast<R *>(x->ws + x->L.off_jtmp);
        dim3 g((unsigned)x->L.pub.tiles_total), b(256);
        int most = MOST;
        while (most > 0 && filter_lds(x, most) > 64 * 1024) --most;
        int launches = passes;
        if (most > 0 && passes > 1) launches = std::min(passes, 2 * ((passes + 2 * most - 1) / (2 * most)));
        for (int k = 0; k < launches; ++k) {
            const R *src = k % 2 ? tmp : p.J;
            R *dst = k % 2 ? p.J : tmp;
            const int now = passes / launches + (k < passes % launches);
            if (most > 0) {
                const size_t lds = filter_lds(x, now);
                pic_status st = set_lds(pic::k_filter<R, D>, lds);
                if (st) return st;
                hipLaunchKernelGGL((pic::k_filter<R, D>), g, b, lds, x->stream, p, src, dst, now);
            } else {
                hipLaunchKernelGGL((pic::k_filter_direct<R, D>), g, b, 0, x->stream, p, src, dst);
            }
        }
        if (launches % 2) {
            const int64_t n = 3 * x->L.pub.cells_total;
            hipLaunchKernelGGL((pic::k_copy<R>), dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), b, 0,
                               x->stream, p.J, tmp, n);
        }
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    static pic_status unpermute(pic_ctx *x, const void *la, const void *ua, void *lb, void *ub, int64_t stride)
    {
        Params<R> p = params<R>(x);
        int64_t maxcap = 1;
        for (int32_t c : x->L.seg_cap) maxcap = std::max<int64_t>(maxcap, c);
        const dim3 grid((unsigned)(x->L.pub.tiles_total * x->ns), (unsigned)((maxcap + 255) / 256));
        hipLaunchKernelGGL((pic::k_adj_unpermute<R, D>), grid, dim3(256), 0, x->stream, p,
                           reinterpret_cast<const R *>(la), reinterpret_cast<const R *>(ua),
                           reinterpret_cast<R *>(lb), reinterpret_cast<R *>(ub), stride);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // per-tile diagnostic partials into part [tiles][NPART] and the charge
    // blocks into rblk [tiles][(T+1)^D]
    static pic_status diag_partials(pic_ctx *x, double *part, double *rblk, int cont_valid)
    {
        Params<R> p = params<R>(x);
        const Layout &L = x->L;
        const double *mass = reinterpret_cast<const double *>(x->ws + L.off_mass);
        size_t lds = L.rblk_cells * sizeof(double);
        pic_status st = set_lds(pic::k_diag_tile<R, D>, lds);
        if (st) return st;
        dim3 g((unsigned)L.pub.tiles_total);
        hipLaunchKernelGGL((pic::k_diag_tile<R, D>), g, dim3(256), lds, x->stream, p, mass, part, rblk);
        double *rho_prev = reinterpret_cast<double *>(x->ws + L.off_rho_prev);
        hipLaunchKernelGGL((pic::k_diag_gauss<R, D>), g, dim3(256), 0, x->stream, p, part, rblk, rho_prev, cont_valid);
        HIP_OK(hipGetLastError());
        return PIC_OK;
    }

    // the diagnostics with the partials in the static scratch, reduced on
    // the device; no allocation of any kind
    static pic_status diag_static(pic_ctx *x, pic_diag *out)
    {
        const Layout &L = x->L;
        const uint64_t part_bytes = align256(L.pub.tiles_total * pic::NPART * sizeof(double));
        const uint64_t rblk_bytes = align256(L.pub.tiles_total * L.rblk_cells * sizeof(double));
        const uint64_t need = part_bytes + rblk_bytes + align256(sizeof(pic::DiagRec));
        if (need > STATIC_SCRATCH_BYTES)
            return fail(PIC_E_ARG, "pic_diagnostics_static needs %llu bytes of static scratch for %lld tiles; "
                                   "the limit is %llu bytes (use pic_diagnostics)",
                        (unsigned long long)need, (long long)L.pub.tiles_total,
                        (unsigned long long)STATIC_SCRATCH_BYTES);
        double *part = reinterpret_cast<double *>(x->scratch);
        double *rblk = reinterpret_cast<double *>(x->scratch + part_bytes);
        pic::DiagRec *rec = reinterpret_cast<pic::DiagRec *>(x->scratch + part_bytes + rblk_bytes);
        const int cont_valid = x->diag_step >= 0 && x->steps - x->diag_step == 1;
        pic_status st = diag_partials(x, part, rblk, cont_valid);
        if (st) return st;
        hipLaunchKernelGGL(pic::k_diag_reduce, dim3(1), dim3(64), 0, x->stream, part, L.pub.tiles_total, cont_valid,
                           rec);
        HIP_OK(hipGetLastError());
        pic::DiagRec h{};
        HIP_OK(hipMemcpyAsync(&h, rec, sizeof h, hipMemcpyDeviceToHost, x->stream));
        HIP_OK(hipStreamSynchronize(x->stream));
        memset(out, 0, sizeof *out);
        out->field_energy = h.field_energy;
        out->kinetic_energy = h.kinetic_energy;
        out->gauss_max = h.gauss_max;
        out->divb_max = h.divb_max;
        out->charge_total = h.charge_total;
        out->particles = h.particles;
        out->near_face = h.near_face;
        out->continuity_max = h.continuity_max;
        x->diag_step = x->steps;
        return PIC_OK;
    }

    // The partials and the error word come to the host in one wait; copies into
    // page-locked memory queue behind the kernels, others wait one by one
    // (five steps and diagnostics of 512x384 FP32: 613 us with two waits, 566 us).
    static pic_status diag(pic_ctx *x, pic_diag *out, bool per_box, int32_t *bits)
    {
        const Layout &L = x->L;
        double *part = reinterpret_cast<double *>(x->ws + L.off_part);
        double *rblk = reinterpret_cast<double *>(x->ws + L.off_rblk);
        const int cont_valid = x->diag_step >= 0 && x->steps - x->diag_step == 1;
        pic_status st = diag_partials(x, part, rblk, cont_valid);
        if (st) return st;
        const size_t n = (size_t)L.pub.tiles_total * pic::NPART;
        if (!x->pin) x->pin = static_cast<double *>(page_locked((n + 1) * sizeof(double)));
        std::vector<double> own(x->pin ? 0 : n + 1);
        double *h = x->pin ? x->pin : own.data();
        HIP_OK(hipMemcpyAsync(h, part, n * sizeof(double), hipMemcpyDeviceToHost, x->stream));
        HIP_OK(hipMemcpyAsync(h + n, x->ws + L.pub.off_error, sizeof(int32_t), hipMemcpyDeviceToHost, x->stream));
        HIP_OK(hipStreamSynchronize(x->stream));
        memcpy(bits, h + n, sizeof *bits);
        const int nout = per_box ? x->nb : 1;
        memset(out, 0, nout * sizeof *out);
        for (int64_t t = 0; t < L.pub.tiles_total; ++t) {
            const double *o = h + t * pic::NPART;
            pic_diag *d = per_box ? out + L.tiles[t].box : out;
            d->field_energy += o[0];
            d->divb_max = std::max(d->divb_max, o[1]);
            d->kinetic_energy += o[2];
            d->particles += (int64_t)o[3];
            d->gauss_max = std::max(d->gauss_max, o[4]);
            d->charge_total += o[5];
            d->near_face += (int64_t)o[7];
        }
        for (int k = 0; k < nout; ++k) out[k].continuity_max = cont_valid ? 0.0 : -1.0;
        if (cont_valid)
            for (int64_t t = 0; t < L.pub.tiles_total; ++t) {
                pic_diag *d = per_box ? out + L.tiles[t].box : out;
                d->continuity_max = std::max(d->continuity_max, h[t * pic::NPART + 6]);
            }
        x->diag_step = x->steps;
        return PIC_OK;
    }
};

#define PIC_DISPATCH(ctx, CALL)                                      \
    do {                                                             \
        if ((ctx)->prec == PIC_FP32) {                               \
            switch ((ctx)->D) {                                      \
            case 1: return Impl<float, 1>::CALL;                     \
            case 2: return Impl<float, 2>::CALL;                     \
            default: return Impl<float, 3>::CALL;                    \
            }                                                        \
        } else {                                                     \
            switch ((ctx)->D) {                                      \
            case 1: return Impl<double, 1>::CALL;                    \
            case 2: return Impl<double, 2>::CALL;                    \
            default: return Impl<double, 3>::CALL;                   \
            }                                                        \
        }                                                            \
    } while (0)

pic_status do_init(pic_ctx *x, const int64_t *counts, const pic_init_data *in) { PIC_DISPATCH(x, init(x, counts, in)); }
pic_status do_fdtd(pic_ctx *x, int phase) { PIC_DISPATCH(x, fdtd(x, phase)); }
pic_status do_push(pic_ctx *x, bool fused, bool halfb) { PIC_DISPATCH(x, push(x, fused, halfb)); }
pic_status do_deposit(pic_ctx *x, bool unfused, bool curl_e) { PIC_DISPATCH(x, deposit(x, unfused, curl_e)); }
pic_status do_finish_step(pic_ctx *x) { PIC_DISPATCH(x, finish_step(x)); }
pic_status do_migrate(pic_ctx *x, bool out, bool in, bool sort, int32_t *mc, int64_t *fl, int64_t fcap)
{
    PIC_DISPATCH(x, migrate(x, out, in, sort, mc, fl, fcap));
}
pic_status do_finish_rows(pic_ctx *x, bool two_halves) { PIC_DISPATCH(x, finish_rows(x, two_halves)); }
pic_status do_diag(pic_ctx *x, pic_diag *o, bool per_box, int32_t *bits) { PIC_DISPATCH(x, diag(x, o, per_box, bits)); }
pic_status do_diag_static(pic_ctx *x, pic_diag *o) { PIC_DISPATCH(x, diag_static(x, o)); }
pic_status do_adjoint(pic_ctx *x, void *a, void *b, void *c, void *d, const void *im, void *op, void *ou, int64_t os)
{
    PIC_DISPATCH(x, adjoint(x, a, b, c, d, im, op, ou, os));
}
pic_status do_state_bytes(pic_ctx *x, uint64_t *out) { PIC_DISPATCH(x, state_bytes(x, out)); }
pic_status do_state_copy(pic_ctx *x, void *image, bool save) { PIC_DISPATCH(x, state_copy(x, image, save)); }
pic_status do_filter(pic_ctx *x, int passes) { PIC_DISPATCH(x, filter(x, passes)); }
pic_status do_inject(pic_ctx *x, int b, int s, int64_t n, const double *pos, const double *u)
{
    PIC_DISPATCH(x, inject(x, b, s, n, pos, u));
}
pic_status do_unpermute(pic_ctx *x, const void *a, const void *b, void *c, void *d, int64_t s)
{
    PIC_DISPATCH(x, unpermute(x, a, b, c, d, s));
}

template <typename R>
pic_status upload_tables(pic_ctx *x, const pic_config *cfg)
{
    const Layout &L = x->L;
    uint8_t *ws = x->ws;
    const int n = x->nb * x->ns;
    std::vector<R> ch(n), qm(n);
    for (int i = 0; i < n; ++i) {
        ch[i] = (R)cfg->charge[i];
        qm[i] = (R)cfg->qm[i];
    }
    x->mass.assign(cfg->mass, cfg->mass + n);
    HIP_OK(hipMemcpy(ws + L.off_charge, ch.data(), n * sizeof(R), hipMemcpyHostToDevice));
    HIP_OK(hipMemcpy(ws + L.off_qm, qm.data(), n * sizeof(R), hipMemcpyHostToDevice));
    return PIC_OK;
}

pic_status clear_error(pic_ctx *x)
{
    pic_status st = fill<int32_t>(x, reinterpret_cast<int32_t *>(x->ws + x->L.pub.off_error), 1, 0);
    if (st) return st;
    HIP_OK(hipStreamSynchronize(x->stream));
    return PIC_OK;
}

pic_status read_error(pic_ctx *x, int32_t *bits)
{
    int32_t *err = reinterpret_cast<int32_t *>(x->ws + x->L.pub.off_error);
    HIP_OK(hipMemcpyAsync(bits, err, sizeof(int32_t), hipMemcpyDeviceToHost, x->stream));
    HIP_OK(hipStreamSynchronize(x->stream));
    return *bits ? clear_error(x) : PIC_OK;
}

pic_status error_status(int32_t bits)
{
    pic_status st = 0;
    if (bits & pic::ERR_CAPACITY) st |= PIC_E_CAPACITY;
    if (bits & pic::ERR_CFL) st |= PIC_E_CFL;
    if (bits & pic::ERR_NONFINITE) st |= PIC_E_NONFINITE;
    if (bits & pic::ERR_OUT_OF_TILE) st |= PIC_E_OUT_OF_TILE;
    if (bits & pic::ERR_ADJ_MAP) st |= PIC_E_ADJ_MAP;
    if (st) fail(st, "device error bits 0x%x", bits);
    return st;
}

}  // namespace

extern "C" {

pic_status pic_query(const pic_config *cfg, const int64_t *counts, pic_layout *out)
{
    if (!out) return fail(PIC_E_ARG, "null output");
    Layout L;
    pic_status st = make_layout(cfg, counts, L);
    if (st) return st;
    *out = L.pub;
    return PIC_OK;
}

pic_status pic_init_tiles(const pic_config *cfg, const int64_t *counts, void *workspace, uint64_t workspace_bytes,
                          const pic_init_data *init, void *hip_stream, pic_ctx **out)
{
    if (!out || !init) return fail(PIC_E_ARG, "null argument");
    *out = nullptr;
    pic_ctx *x = new pic_ctx();
    pic_status st = make_layout(cfg, counts, x->L);
    if (st) {
        delete x;
        return st;
    }
    if (!workspace || workspace_bytes < x->L.pub.total_bytes || (reinterpret_cast<uintptr_t>(workspace) & 255)) {
        delete x;
        return fail(PIC_E_ARG, "workspace must be 256-byte aligned and hold %llu bytes",
                    (unsigned long long)x->L.pub.total_bytes);
    }
    x->D = cfg->dim;
    x->prec = cfg->precision;
    x->ns = cfg->n_species;
    x->nb = cfg->n_boxes;
    x->block = cfg->block ? cfg->block : 256;
    x->acc_working = (cfg->options & PIC_OPT_ACC_WORKING) != 0;
    x->persistent = (cfg->options & PIC_OPT_PERSISTENT) != 0;
    x->track = (cfg->options & PIC_OPT_TRACK) != 0;
    x->exact_block = (cfg->options & PIC_OPT_EXACT_BLOCK) != 0;
    x->walls = false;
    x->pusher = cfg->pusher;
    x->filter_passes = cfg->filter_passes;
    x->order = cfg->fdtd_order == 4 ? 4 : 2;
    x->steps = 0;
    x->order_age = ORDER_EVERY;
    x->diag_step = -1;
    x->pin = nullptr;
    for (int b = 0; cfg->box_walls && b < cfg->n_boxes; ++b) x->walls = x->walls || (cfg->box_walls[b] & PIC_WALL_X);
    x->graph = nullptr;
    x->graph_steps = 0;
    {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
            delete x;
            return fail(PIC_E_HIP, "cannot query the device");
        }
        x->n_cu = prop.multiProcessorCount;
        x->push_group[0] = x->push_group[1] = 0;
    }
    for (int d = 0; d < 3; ++d) x->T[d] = cfg->tile[d];
    x->c = cfg->cfl;
    x->stream = reinterpret_cast<hipStream_t>(hip_stream);
    x->ws = reinterpret_cast<uint8_t *>(workspace);
    x->state = 0;
    x->all_species = (1u << x->ns) - 1u;
    x->pushed = 0;
    x->launch_mask = x->all_species;
    x->step_b = false;
    const Layout &L = x->L;
    auto cleanup = [&](pic_status s) {
        delete x;
        return s;
    };
#define INIT_HIP(expr)                                                                           \
    do {                                                                                         \
        hipError_t e_ = (expr);                                                                  \
        if (e_ != hipSuccess) return cleanup(fail(PIC_E_HIP, "%s: %s", #expr, hipGetErrorString(e_))); \
    } while (0)
    INIT_HIP(hipStreamSynchronize(x->stream));
    {
        void *sp = nullptr;
        if ((st = scratch_address(&sp))) return cleanup(st);
        x->scratch = reinterpret_cast<uint8_t *>(sp);
    }
    INIT_HIP(hipMemcpy(x->ws + L.off_tiles, L.tiles.data(), L.tiles.size() * sizeof(TileDesc), hipMemcpyHostToDevice));
    INIT_HIP(hipMemcpy(x->ws + L.pub.off_seg_offset, L.seg_off.data(), L.seg_off.size() * 8, hipMemcpyHostToDevice));
    INIT_HIP(hipMemcpy(x->ws + L.pub.off_seg_capacity, L.seg_cap.data(), L.seg_cap.size() * 4, hipMemcpyHostToDevice));
    INIT_HIP(hipMemcpy(x->ws + L.off_order, L.order.data(), L.order.size() * 4, hipMemcpyHostToDevice));
    INIT_HIP(hipMemcpy(x->ws + L.off_mass, cfg->mass, (size_t)x->nb * x->ns * 8, hipMemcpyHostToDevice));
    st = x->prec == PIC_FP32 ? upload_tables<float>(x, cfg) : upload_tables<double>(x, cfg);
    if (st) return cleanup(st);
    if ((st = fill<int32_t>(x, reinterpret_cast<int32_t *>(x->ws + L.pub.off_error), 1, 0))) return cleanup(st);
    if ((st = do_init(x, counts, init))) return cleanup(st);
    int32_t bits = 0;
    if ((st = read_error(x, &bits))) return cleanup(st);
    if (bits) return cleanup(error_status(bits));
#undef INIT_HIP
    *out = x;
    return PIC_OK;
}

pic_status pic_fdtd_step(pic_ctx *x, int32_t phase)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    return do_fdtd(x, phase);
}

// species mask of a push or deposit call: PIC_ALL_SPECIES or a nonempty
// subset of the context's species
static pic_status species_of(pic_ctx *x, uint32_t mask, uint32_t *out)
{
    if (mask == PIC_ALL_SPECIES) mask = x->all_species;
    if (!mask || (mask & ~x->all_species))
        return fail(PIC_E_ARG, "species mask 0x%x: empty or beyond the %d species", mask, x->ns);
    if (x->track && mask != x->all_species)
        return fail(PIC_E_ARG, "origin tracking (PIC_OPT_TRACK) needs every species in one call");
    *out = mask;
    return PIC_OK;
}

pic_status pic_push_interp(pic_ctx *x, uint32_t species_mask, uint32_t flags)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    uint32_t mask = 0;
    pic_status st = species_of(x, species_mask, &mask);
    if (st) return st;
    const bool fused = flags & PIC_FUSED;
    if (x->state >= 3) return fail(PIC_E_STATE, "push called after this step's deposit");
    if (x->state != 0 && (x->state == 2) != fused)
        return fail(PIC_E_STATE, "every push of a step must use the same PIC_FUSED setting");
    if (x->pushed & mask) return fail(PIC_E_STATE, "species 0x%x already pushed in this step", x->pushed & mask);
    if (x->order == 4 && (flags & PIC_PUSH_HALF_B))
        return fail(PIC_E_ARG, "PIC_PUSH_HALF_B applies the second-order half update; use pic_fdtd_step with FDTD4");
    if (x->track && !fused) return fail(PIC_E_ARG, "origin tracking records origins in the fused push only");
    if (x->walls && !fused) return fail(PIC_E_ARG, "boxes with walls need the fused push (PIC_FUSED)");
    x->launch_mask = mask;
    st = do_push(x, fused, (flags & PIC_PUSH_HALF_B) != 0);
    x->launch_mask = x->all_species;
    if (st) return st;
    x->pushed |= mask;
    x->state = fused ? 2 : 1;
    return PIC_OK;
}

pic_status pic_push_threads(pic_ctx *x, uint32_t flags, int32_t *threads)
{
    if (!x || !threads) return fail(PIC_E_ARG, "null argument");
    *threads = x->push_group[(flags & PIC_FUSED) != 0];
    return PIC_OK;
}

pic_status pic_deposit_current(pic_ctx *x, uint32_t species_mask, uint32_t flags)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    uint32_t mask = 0;
    pic_status st = species_of(x, species_mask, &mask);
    if (st) return st;
    const bool curl_e = flags & PIC_DEPOSIT_CURL_E;
    if (curl_e && x->order != 2) return fail(PIC_E_ARG, "PIC_DEPOSIT_CURL_E applies the second-order E update; use pic_fdtd_step with FDTD4");
    if (x->state != 1 && x->state != 2) return fail(PIC_E_STATE, "deposit needs a preceding push (once per step)");
    if (mask & ~x->pushed) return fail(PIC_E_STATE, "species 0x%x not pushed in this step", mask & ~x->pushed);
    x->launch_mask = mask;
    st = do_deposit(x, x->state == 1, curl_e);
    x->launch_mask = x->all_species;
    if (st) return st;
    x->state = 3 + (x->state == 2 ? 1 : 0);   // 3: unfused deposited, 4: fused deposited
    return PIC_OK;
}

pic_status pic_sort_migrate(pic_ctx *x, uint32_t flags, int32_t *migration_counts, int64_t *flagged,
                            int64_t flagged_capacity)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    if (x->state == 1) return fail(PIC_E_STATE, "deposit the current of an unfused push before migrating");
    if (flagged_capacity < 0) return fail(PIC_E_ARG, "flagged_capacity must be >= 0");
    const bool sort = flags & PIC_SORT_CELLS;
    if (x->track && sort) return fail(PIC_E_ARG, "the cell sort does not record origins (PIC_OPT_TRACK)");
    const bool stepped = x->state != 0;
    if (migration_counts && !stepped) return fail(PIC_E_STATE, "migration counts need a preceding push");
    pic_status st;
    if (x->state == 3) st = do_migrate(x, true, true, sort, migration_counts, flagged, flagged_capacity);
    else if (stepped) st = do_migrate(x, false, true, sort, migration_counts, flagged, flagged_capacity);
    else st = do_migrate(x, false, false, sort, nullptr, flagged, flagged_capacity);   // nothing moved
    if (st) return st;
    x->state = 0;
    x->pushed = 0;
    if (stepped) ++x->steps;
    return PIC_OK;
}

// deposit (or fold), filter, E += c curl- B - J; with FDTD2 and no filter
// the fold and the E update are one pass.
static pic_status current_and_e(pic_ctx *x, uint32_t flags)
{
    pic_status st;
    if (!x->filter_passes && x->order == 2) return pic_deposit_current(x, PIC_ALL_SPECIES, flags | PIC_DEPOSIT_CURL_E);
    if ((st = pic_deposit_current(x, PIC_ALL_SPECIES, flags))) return st;
    if (x->filter_passes && (st = pic_filter_current(x, x->filter_passes))) return st;
    return pic_fdtd_step(x, PIC_CURL_E_ADD_J);
}

// After the last row of a fused step: the arrivals are in.
static pic_status end_step(pic_ctx *x, uint32_t flags)
{
    x->state = 0;
    x->pushed = 0;
    ++x->steps;
    return flags & PIC_SORT_CELLS ? do_migrate(x, false, false, true, nullptr, nullptr, 0) : PIC_OK;
}

pic_status pic_step(pic_ctx *x, uint32_t flags)
{
    pic_status st;
    if (!x) return fail(PIC_E_ARG, "null context");
    if (x->order == 4) flags &= ~PIC_PUSH_HALF_B;   // the in-LDS half update is second order
    flags &= ~PIC_DEPOSIT_CURL_E;                    // chosen below
    const bool untracked_sort = x->track && (flags & PIC_SORT_CELLS);   // refused by pic_sort_migrate
    const bool rows =
        (flags & PIC_FUSED) && (x->order == 4 || x->filter_passes) && x->state == 0 && !untracked_sort;
    if (flags & PIC_PUSH_HALF_B) {
        if ((flags & PIC_FUSED) && x->order == 2 && !x->filter_passes && x->state == 0 && !untracked_sort) {
            // two launches: the push, which also leaves B after both half
            // updates in the filter's scratch planes, and the rest of the
            // step.  After the push, half B, fold with E and migration as
            // launches of their own took 12.6 us (1D, 512 cells FP64), 17 us
            // (2D 256^2 FP32), 69 us (2D 1024^2 FP32) and 126 us (3D
            // 256x64x64 with walls FP32), the one launch 4.0, 5.9, 54.6 and
            // 89 us.
            x->step_b = true;
            st = pic_push_interp(x, PIC_ALL_SPECIES, flags);
            x->step_b = false;
            if (st || (st = do_finish_step(x))) return st;
            return end_step(x, flags);
        }
        // push_half_b1 happens inside the push on its LDS copy of B; both
        // half updates are then applied to the stored B in one pass
        if ((st = pic_push_interp(x, PIC_ALL_SPECIES, flags))) return st;
        if (rows) return (st = do_finish_rows(x, true)) ? st : end_step(x, flags);
        if ((st = pic_fdtd_step(x, PIC_TWO_HALF_B))) return st;
        if ((st = current_and_e(x, flags))) return st;
        return pic_sort_migrate(x, flags, nullptr, nullptr, 0);
    }
    if ((st = pic_fdtd_step(x, PIC_HALF_B))) return st;
    if ((st = pic_push_interp(x, PIC_ALL_SPECIES, flags))) return st;
    if (rows) return (st = do_finish_rows(x, false)) ? st : end_step(x, flags);
    if ((st = pic_fdtd_step(x, PIC_HALF_B))) return st;
    if ((st = current_and_e(x, flags))) return st;
    return pic_sort_migrate(x, flags, nullptr, nullptr, 0);
}

pic_status pic_inject(pic_ctx *x, int32_t box, int32_t species, int64_t count, const double *pos, const double *u)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    if (x->state != 0) return fail(PIC_E_STATE, "inject between steps");
    if (box < 0 || box >= x->nb || species < 0 || species >= x->ns) return fail(PIC_E_ARG, "box or species out of range");
    if (count < 0 || count > x->L.max_count)
        return fail(PIC_E_ARG, "a batch holds at most %lld particles (pic_config.inject_max)", (long long)x->L.max_count);
    if (count == 0) return PIC_OK;
    if (!pos || !u) return fail(PIC_E_ARG, "pos and u are required");
    x->order_age = ORDER_EVERY;   // counts changed: re-sort at the next push
    return do_inject(x, box, species, count, pos, u);
}

pic_status pic_filter_current(pic_ctx *x, int32_t passes)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    if (passes < 0) return fail(PIC_E_ARG, "passes must be >= 0");
    if (x->walls) return fail(PIC_E_ARG, "the current filter covers periodic boxes only");
    if (passes == 0) return PIC_OK;
    return do_filter(x, passes);
}

pic_status pic_graph_capture(pic_ctx *x, int32_t nsteps, uint32_t flags)
{
    if (!x || nsteps < 1) return fail(PIC_E_ARG, "need a context and nsteps >= 1");
    if (x->state != 0) return fail(PIC_E_STATE, "capture must start between steps");
    if (!x->stream) return fail(PIC_E_ARG, "graph capture needs a context on a created (non-default) stream");
    if (x->graph) {
        HIP_OK(hipGraphExecDestroy(x->graph));
        x->graph = nullptr;
    }
    // one eager step sets the kernels' LDS attributes before capture
    pic_status st = pic_step(x, flags);
    if (st) return st;
    HIP_OK(hipStreamSynchronize(x->stream));
    const int64_t steps_before = x->steps;   // captured steps do not run now
    HIP_OK(hipStreamBeginCapture(x->stream, hipStreamCaptureModeThreadLocal));
    // the first captured push takes a new order, a later eager one too (replays
    // change the counts)
    x->order_age = ORDER_EVERY;
    for (int k = 0; k < nsteps && !st; ++k) st = pic_step(x, flags);
    x->order_age = ORDER_EVERY;
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(x->stream, &g);
    x->steps = steps_before;
    if (st) {
        if (g) (void)hipGraphDestroy(g);
        return st;
    }
    if (e != hipSuccess) return fail(PIC_E_HIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
    e = hipGraphInstantiate(&x->graph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
        x->graph = nullptr;
        return fail(PIC_E_HIP, "hipGraphInstantiate: %s", hipGetErrorString(e));
    }
    x->graph_steps = nsteps;
    return PIC_OK;
}

pic_status pic_graph_launch(pic_ctx *x)
{
    if (!x || !x->graph) return fail(PIC_E_STATE, "no captured graph");
    HIP_OK(hipGraphLaunch(x->graph, x->stream));
    x->steps += x->graph_steps;
    return PIC_OK;
}

pic_status pic_error(pic_ctx *x)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    int32_t bits = 0;
    pic_status st = read_error(x, &bits);
    if (st) return st;
    return error_status(bits);
}

pic_status pic_diagnostics(pic_ctx *x, pic_diag *out)
{
    if (!x || !out) return fail(PIC_E_ARG, "null argument");
    int32_t bits = 0;
    pic_status st = do_diag(x, out, false, &bits);
    if (st || (bits && (st = clear_error(x)))) return st;
    out->error_bits = bits;
    return error_status(bits);
}

pic_status pic_diagnostics_static(pic_ctx *x, pic_diag *out)
{
    if (!x || !out) return fail(PIC_E_ARG, "null argument");
    pic_status st = do_diag_static(x, out);
    if (st) return st;
    int32_t bits = 0;
    if ((st = read_error(x, &bits))) return st;
    out->error_bits = bits;
    return error_status(bits);
}

pic_status pic_diagnostics_boxes(pic_ctx *x, pic_diag *out)
{
    if (!x || !out) return fail(PIC_E_ARG, "null argument");
    int32_t bits = 0;
    pic_status st = do_diag(x, out, true, &bits);
    if (st || (bits && (st = clear_error(x)))) return st;
    for (int b = 0; b < x->nb; ++b) out[b].error_bits = bits;
    return error_status(bits);
}

pic_status pic_adjoint_unpermute(pic_ctx *x, const void *lpos_after, const void *lu_after, void *lpos_before,
                                 void *lu_before, int64_t before_stride)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    if (!x->track) return fail(PIC_E_STATE, "the context was created without PIC_OPT_TRACK");
    if (!lpos_after || !lu_after || !lpos_before || !lu_before || before_stride < 1)
        return fail(PIC_E_ARG, "adjoint buffers and a positive before_stride are required");
    if (x->state != 0) return fail(PIC_E_STATE, "unpermute must run between steps");
    return do_unpermute(x, lpos_after, lu_after, lpos_before, lu_before, before_stride);
}

static pic_status adjoint_checks(pic_ctx *x, const void *lpos, const void *lu, const void *lE, const void *lB)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    if (!x->track) return fail(PIC_E_STATE, "the context was created without PIC_OPT_TRACK");
    if (x->walls) return fail(PIC_E_ARG, "the adjoint step covers periodic boxes only");
    if (x->pusher != PIC_PUSHER_BORIS || x->filter_passes || x->order != 2)
        return fail(PIC_E_ARG, "the adjoint step covers the Boris pusher and FDTD2 without current filter");
    if (!lpos || !lu || !lE || !lB) return fail(PIC_E_ARG, "adjoint buffers are required");
    if (x->state != 0) return fail(PIC_E_STATE, "the adjoint step must start between steps");
    return PIC_OK;
}

pic_status pic_adjoint_step(pic_ctx *x, void *lpos, void *lu, void *lE, void *lB)
{
    pic_status st = adjoint_checks(x, lpos, lu, lE, lB);
    return st ? st : do_adjoint(x, lpos, lu, lE, lB, nullptr, nullptr, nullptr, 0);
}

pic_status pic_adjoint_reverse(pic_ctx *x, const void *image, void *lpos, void *lu, void *lE, void *lB,
                               void *lpos_before, void *lu_before, int64_t before_stride)
{
    pic_status st = adjoint_checks(x, lpos, lu, lE, lB);
    if (st) return st;
    if (!lpos_before || !lu_before || before_stride < 1)
        return fail(PIC_E_ARG, "the adjoints' destination and a positive before_stride are required");
    // tiles store to the destination while others still read lpos and lu
    const uint64_t w = x->prec == PIC_FP64 ? 8 : 4, cap = (uint64_t)x->L.pub.capacity_total * w, out = (uint64_t)before_stride * w;
    auto overlap = [](const void *a, uint64_t na, const void *b, uint64_t nb) {
        const uint64_t p = reinterpret_cast<uintptr_t>(a), q = reinterpret_cast<uintptr_t>(b);
        return p < q + nb && q < p + na;
    };
    if (overlap(lpos, x->D * cap, lpos_before, x->D * out) || overlap(lpos, x->D * cap, lu_before, 3 * out) ||
        overlap(lu, 3 * cap, lpos_before, x->D * out) || overlap(lu, 3 * cap, lu_before, 3 * out) ||
        overlap(lpos_before, x->D * out, lu_before, 3 * out))
        return fail(PIC_E_ARG, "the particle adjoints and their destination must not overlap");
    if (reinterpret_cast<uintptr_t>(image) & 255) return fail(PIC_E_ARG, "a state image must be 256-byte aligned");
    return do_adjoint(x, lpos, lu, lE, lB, image, lpos_before, lu_before, before_stride);
}

static pic_status image_checks(pic_ctx *x, const void *image)
{
    if (!x) return fail(PIC_E_ARG, "null context");
    if (!x->track) return fail(PIC_E_STATE, "the context was created without PIC_OPT_TRACK");
    if (x->state != 0) return fail(PIC_E_STATE, "states are saved and loaded between steps");
    if (!image || (reinterpret_cast<uintptr_t>(image) & 255)) return fail(PIC_E_ARG, "a state image must be 256-byte aligned");
    return PIC_OK;
}

pic_status pic_state_bytes(pic_ctx *x, uint64_t *bytes)
{
    if (!x || !bytes) return fail(PIC_E_ARG, "null argument");
    return do_state_bytes(x, bytes);
}

pic_status pic_state_save(pic_ctx *x, void *image)
{
    pic_status st = image_checks(x, image);
    return st ? st : do_state_copy(x, image, true);
}

pic_status pic_state_load(pic_ctx *x, const void *image)
{
    pic_status st = image_checks(x, image);
    if (st || (st = do_state_copy(x, const_cast<void *>(image), false))) return st;
    x->diag_step = -1;   // the last diagnostics were of another state: no continuity from them
    return PIC_OK;
}

pic_status pic_destroy(pic_ctx *x)
{
    if (x && x->graph) (void)hipGraphExecDestroy(x->graph);
    if (x && x->pin) free_page_locked(x->pin);
    delete x;
    return PIC_OK;
}

const char *pic_last_error(void) { return g_last_error; }

}  // extern "C"
