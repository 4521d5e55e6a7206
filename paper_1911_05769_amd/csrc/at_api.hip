// Host side of libat.so: configuration checks, workspace layout, delay set-up,
// launch sequencing (plain, fused, recorded), checkpoints, adjoint sweep,
// snapshots, reductions and the autotuner.  See include/at.h for the contract.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <string>
#include <vector>

#include "../../include/at.h"
#include "at_internal.h"

using namespace atk;

// 3D hooks (defined in at_step3d.hip)
at_status at3_check(const at_config *c);
uint64_t at3_ring_level_doubles(const at_config *c);

namespace {

thread_local std::string g_err;

at_status fail(at_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

#define AT_HIP(call)                                                                   \
    do {                                                                               \
        hipError_t e_ = (call);                                                        \
        if (e_ != hipSuccess)                                                          \
            return fail(AT_ERR_HIP, "%s failed: %s", #call, hipGetErrorString(e_));    \
    } while (0)

constexpr uint64_t kAlign = 256;
constexpr int kWholeVariant = 4;   // 1D: the whole grid in one workgroup
uint64_t align_up(uint64_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Layout {
    uint64_t delays = 0, ring = 0, red = 0, sync = 0, ckpt = 0, seg = 0, lam = 0, mu = 0, gnu = 0,
             total = 0;
    int64_t nckpt = 0, ngnu = 0;
    int R = 0, Rmu = 0;
};

struct Derived {
    int dim, order, h, m;
    int L;          // delay bound
    int fppt = 16;  // 1D: points per thread of the regions that limit steps per launch
    int64_t N;      // total points
    int64_t F;      // faces
    int64_t nb;     // tiles / blocks
    int64_t P, W;   // 1D
    double c1[3], c2[3];
    bool contracted = false;
};

// Region of a workgroup of 256 threads: RL points left of the owned chunk, CH
// owned, s*h right; where the tile width is a multiple of the points per
// thread, RL and CH are multiples of it too.  The one-step and the general
// kernel run these, and region_limit measures with them what at_set_fuse
// accepts (a launch of the fused kernels takes as many of those steps as its
// own region allows, launch_steps).
struct Region1D {
    int ppt;        // points per thread
    int64_t RL, CH;
};

// Points per thread that region_limit's regions are measured at: the most (16,
// 8, 4) that still give every SIMD four waves of the grid and divide the tile
// width; 16 when none divides it
int fused_ppt(const Derived &d)
{
    const int opts[3] = {16, 8, 4};
    int pick = 0;
    for (int i = 0; i < 3; ++i) {
        const int p = opts[i];
        if (d.W % p != 0) continue;
        if (pick == 0) pick = p;
        if (d.N >= (int64_t)4 * 1024 * 64 * p) return p;
        pick = p;
    }
    return pick ? pick : 16;
}

at_status derive(const at_config *c, Derived &d)
{
    if (!c) return fail(AT_ERR_ARG, "null configuration");
    if (c->abi_version != AT_ABI_VERSION)
        return fail(AT_ERR_ARG, "abi_version %d, library has %d", c->abi_version, AT_ABI_VERSION);
    if (c->dim != 1 && c->dim != 3) return fail(AT_ERR_ARG, "dim must be 1 or 3");
    if (c->order != 2 && c->order != 4) return fail(AT_ERR_ARG, "order must be 2 or 4");
    if (c->dim == 3 && c->order != 2) return fail(AT_ERR_ARG, "3D stepper is order 2");
    if (c->L < 0 || c->L > 15) return fail(AT_ERR_ARG, "L must be in 0..15");
    if (c->halo_mode != 0 && c->halo_mode != 1) return fail(AT_ERR_ARG, "halo_mode must be 0 or 1");
    if (c->adv_mode != 0 && c->adv_mode != 1) return fail(AT_ERR_ARG, "adv_mode must be 0 or 1");
    if (c->adv_mode == 1 && c->dim != 1) return fail(AT_ERR_ARG, "linear advection is 1D only");
    if (!(c->nu >= 0.0) || !isfinite(c->nu)) return fail(AT_ERR_ARG, "nu must be finite and >= 0");
    if (!(c->dt > 0.0) || !isfinite(c->dt)) return fail(AT_ERR_ARG, "dt must be finite and > 0");
    if (!(c->length > 0.0) || !isfinite(c->length)) return fail(AT_ERR_ARG, "length must be > 0");
    if (c->nsteps_max < 0) return fail(AT_ERR_ARG, "nsteps_max must be >= 0");
    if (c->delay_mode != AT_DELAY_GENERATE && c->delay_mode != AT_DELAY_HOST)
        return fail(AT_ERR_ARG, "unknown delay_mode");
    if (c->delay_mode == AT_DELAY_GENERATE && c->delay_dist != AT_DIST_UNIFORM &&
        c->delay_dist != AT_DIST_HALF_ZERO)
        return fail(AT_ERR_ARG, "unknown delay_dist");
    if (c->delay_mode == AT_DELAY_HOST && !c->delays_host && c->nsteps_max > 0)
        return fail(AT_ERR_ARG, "delays_host is NULL");
    if (c->fuse_steps < 0 || c->fuse_steps > kMaxFuse)
        return fail(AT_ERR_ARG, "fuse_steps must be in 0..%d", kMaxFuse);
    if (c->arith != 0 && c->arith != 1) return fail(AT_ERR_ARG, "arith must be 0 or 1");
    if (c->arith == 1 && c->dim != 1) return fail(AT_ERR_ARG, "arith 1 is 1D only");
    if (c->reserved1 != 0) return fail(AT_ERR_ARG, "reserved1 must be 0");
    if (c->nscalars < 0 || c->nscalars > AT_MAX_SCALARS)
        return fail(AT_ERR_ARG, "nscalars must be in 0..%d", AT_MAX_SCALARS);
    if (c->nscalars > 0 && c->dim != 3) return fail(AT_ERR_ARG, "passive scalars are 3D only");
    for (int s = 0; s < c->nscalars; ++s)
        if (!(c->alpha[s] >= 0.0) || !isfinite(c->alpha[s]))
            return fail(AT_ERR_ARG, "alpha[%d] must be finite and >= 0", s);
    if (c->record) {
        if (c->dim != 1) return fail(AT_ERR_ARG, "record mode (adjoint) is 1D only");
        if (c->ckpt_every < 1) return fail(AT_ERR_ARG, "record mode needs ckpt_every >= 1");
    }
    d.dim = c->dim;
    d.order = c->order;
    d.h = c->order / 2;
    d.m = (c->order == 2) ? 2 : 3;
    d.L = c->L;
    const int naxes = c->dim;
    d.N = 1;
    d.nb = 1;
    for (int a = 0; a < 3; ++a) {
        const int64_t n = c->n[a];
        const int64_t p = c->p[a];
        if (a >= naxes) {
            if (n != 1 || p != 1) return fail(AT_ERR_SHAPE, "unused axis %d must have n = p = 1", a);
            d.c1[a] = d.c2[a] = 0.0;
            continue;
        }
        if (n <= 0 || p <= 0) return fail(AT_ERR_SHAPE, "axis %d: n and p must be positive", a);
        if (n % p != 0) return fail(AT_ERR_SHAPE, "axis %d: n %% p != 0", a);
        if (n / p < 2 * d.h) return fail(AT_ERR_SHAPE, "axis %d: tile width %lld < 2h", a,
                                         (long long)(n / p));
        const double dx = c->length / (double)n;
        if (c->order == 2) { d.c1[a] = 1.0 / (2.0 * dx); d.c2[a] = 1.0 / (dx * dx); }
        else { d.c1[a] = 1.0 / (12.0 * dx); d.c2[a] = 1.0 / (12.0 * (dx * dx)); }
        d.N *= n;
        d.nb *= p;
    }
    d.F = (c->dim == 1 ? 2 : 6) * d.nb;
    d.P = c->p[0];
    d.W = c->n[0] / c->p[0];
    if (d.N > ((int64_t)1 << 40)) return fail(AT_ERR_SHAPE, "grid too large");
    if (c->dim == 3) {
        at_status st = at3_check(c);
        if (st != AT_OK) return st;
    }
    d.contracted = c->arith == 1;
    if (d.dim == 1) d.fppt = fused_ppt(d);
    return AT_OK;
}

int max_fuse_1d(const Derived &d);

// ring levels: L+m-1 past levels are read while up to s levels are written
// (s = the largest steps-per-launch this grid allows); record mode keeps every
// level of the run (the adjoint re-reads them).
int ring_levels(const at_config *c, const Derived &d)
{
    // 1D: any steps-per-launch and points-per-thread choice; 3D: a step reads
    // levels n-L-1 .. n and publishes level n+1, and in the weakly-synchronous
    // run a face neighbour up to L steps behind still reads levels down to
    // n-2L-1 while this block writes level n+1: 2L + m + 2 slots keep them apart
    const int smax = d.dim == 1 ? kMaxFuse : c->L + 3;
    int64_t R = c->L + d.m - 1 + smax;
    if (c->record) R = std::max<int64_t>(R, c->nsteps_max + 1);
    return (int)R;
}

}  // namespace

struct at_ctx {
    at_config cfg;
    Derived d;
    Layout lay;
    hipStream_t st;
    int8_t *delays;
    double *ring, *red, *ckpt, *seg, *lam, *mu, *gnu;
    int32_t *sync;   // weakly-synchronous run: level counters (3D: [blocks]), then the error flag
    int64_t n;
    int fuse;
    int variant;     // 3D kernel variant (tile rows, prefetch depth, register budget)
    int32_t brick[4] = {0, 0, 0, 0};   // 3D: brick of the general kernel (0: not picked yet)
    int kind = 0;    // 1D: the variant's region kind (variant_kind), 0 by the estimate
    int adj_fuse = 0;   // reverse steps per adjoint launch: 0 automatic, 1 one-step kernel
    int debug = 0;      // AT_DEBUG_* flags (at_set_debug)
    // graph replay of at_run (at_set_graph): the launch sequence of one call,
    // captured on a private stream and replayed on the context's stream
    int use_graph = 0;
    hipStream_t cap = nullptr;
    hipGraphExec_t gexec = nullptr;
    int64_t g_n0 = -1, g_nsteps = -1;
    const double *g_u = nullptr, *g_s = nullptr;
    int g_fuse = 0, g_variant = -1, g_debug = -1;
    // snapshots taken through this context: device buffer and its step
    std::vector<std::pair<const void *, int64_t>> snaps;
};

namespace {

uint64_t ring_level_doubles(const at_config *c, const Derived &d)
{
    if (d.dim == 1) return (uint64_t)d.P * 2 * d.h;
    return at3_ring_level_doubles(c);
}

int64_t adj_blocks(const Derived &d)
{
    const int64_t per = adj1d_points_per_block();
    return (d.N + per - 1) / per;
}

at_status make_layout(const at_config *c, const Derived &d, Layout &L)
{
    L.R = ring_levels(c, d);
    L.Rmu = c->L + d.m + kMaxFuse;   // levels a fused reverse launch writes and reads stay distinct
    uint64_t off = 0;
    L.delays = off;
    off = align_up(off + (uint64_t)c->nsteps_max * (uint64_t)d.F);
    L.ring = off;
    off = align_up(off + 8ull * (uint64_t)L.R * ring_level_doubles(c, d));
    L.red = off;
    off = align_up(off + 8ull * (kRedBlocks * 6 + 16));
    // level counters of the weakly-synchronous run (3D: one per block; in 1D the
    // edge values tell their arrival themselves), then its error flag
    L.sync = off;
    off = align_up(off + 4ull * ((d.dim == 1 ? 0 : (uint64_t)d.nb) + 64));
    if (c->record) {
        L.nckpt = c->nsteps_max / c->ckpt_every + 1;
        L.ckpt = off;
        off = align_up(off + 8ull * (uint64_t)L.nckpt * (uint64_t)d.N);
        L.seg = off;
        off = align_up(off + 8ull * (uint64_t)c->ckpt_every * (uint64_t)d.N);
        L.lam = off;
        off = align_up(off + 8ull * 2 * (uint64_t)d.N);
        L.mu = off;
        off = align_up(off + 8ull * (uint64_t)L.Rmu * (uint64_t)d.P * 2 * d.h);
        // >= the blocks of any reverse launch: chunks of at least 32 lanes of 3 or
        // 4 points (256 points of the one-step kernel)
        L.ngnu = (d.N + 95) / 96;
        L.gnu = off;
        off = align_up(off + 8ull * 2 * (uint64_t)L.ngnu);
    }
    L.total = off;
    return AT_OK;
}

Region1D region_1d(const Derived &d, int s);

// The most steps per launch at_set_fuse accepts, a limit of the interface: in a
// region of 256 threads the owned chunk stays at least half of it (or the whole
// grid), and a table of its tile edges over the s steps and the D = L + m - 1
// levels below fits 64 KiB beside the field's stage.  (On tiles of a few dozen
// points the fused kernels' own regions would take more: order 4, L = 4: 6 here
// at 33 points, 40 there.)
size_t edge_table_bytes(const Derived &d, int s, int NT, int ppt)
{
    const size_t stage = (size_t)kThreads * (ppt + 1) / (ppt >= 16 ? 2 : 1);
    const size_t xch = (size_t)2 * kThreads * d.order;
    const size_t edges = (size_t)(d.L + d.m - 1 + s - 1) * NT * d.order;
    return 8 * (std::max(stage, xch) + edges + ((size_t)s * NT * 2 + 7) / 8);
}

int region_limit(const Derived &d)
{
    int best = 1;
    for (int s = 2; s <= kMaxFuse; ++s) {
        const Region1D rg = region_1d(d, s);
        const int reg = kThreads * rg.ppt;
        if (rg.CH < std::min<int64_t>(reg / 2, d.N)) break;
        const int NT = (int)((reg - 1) / d.W + 2);
        if (edge_table_bytes(d, s, NT, rg.ppt) > 64 * 1024) break;
        best = s;
    }
    return best;
}

// (that of the variant's points per thread, and no less than variant 0's, whose
// steps at_autotune may choose with any variant)
int max_fuse_1d(const Derived &d)
{
    Derived own = d;
    own.fppt = fused_ppt(d);
    return std::max(region_limit(d), region_limit(own));
}

Region1D region_1d(const Derived &d, int s)
{
    // single steps use the one-step kernel when the tiles allow it
    const int plain = s == 1 ? step1d_plain_ppt(d.W) : 0;
    const int ppt = plain ? plain : (d.W % d.fppt == 0 ? d.fppt : step1d_points_per_thread());
    const int64_t reg = (int64_t)kThreads * ppt;
    Region1D r;
    r.ppt = ppt;
    if (d.W % ppt == 0) {
        r.RL = ((int64_t)s * d.h + ppt - 1) / ppt * ppt;
        r.CH = (reg - r.RL - (int64_t)s * d.h) / ppt * ppt;
    } else {
        r.RL = (int64_t)s * d.h;
        r.CH = reg - 2 * (int64_t)s * d.h;
    }
    if (r.CH > d.N) r.CH = d.N;
    return r;
}

// A region of the fused kernels (at_wave1d.h) for s steps.  kind: the points
// per thread (one of kFusedKinds) of a one-wave region, kWide the four-wave
// region at 16.  ok is false when the tile width is not a sum of threads of ppt and
// ppt - 1 points (a few widths below ppt * (ppt - 2)), when one thread is a
// whole tile, when s is more than the rims allow, or when the LDS tables of
// very narrow tiles exceed 64 KiB.
constexpr int kWide = -16;
constexpr int kFusedKinds[] = {32, 24, 20, 16, 12, 10, 8, 6, 4};

struct FusedShape {
    bool ok = false;
    int ppt = 0, nw = 0, tpt = 0, nf = 0, RT = 0, CT = 0, NT = 0;
    int64_t nblocks = 0;
    size_t lds = 0;
};

FusedShape fused_shape(const Derived &d, int s, int kind)
{
    FusedShape w;
    if (kind == 0 || d.W > ((int64_t)1 << 30)) return w;
    const int ppt = std::abs(kind), nw = kind < 0 ? 4 : 1, threads = 64 * nw;
    const int64_t tpt = (d.W + ppt - 1) / ppt, nf = d.W - tpt * (ppt - 1);
    const int64_t nth = d.P * tpt;
    if (nf < 1 || nth >= ((int64_t)1 << 31) - 256) return w;
    if (kind < 0 && nf != tpt) return w;              // (built for whole threads only)
    if (tpt == 1 && d.W != 4) return w;               // a lane has one face (two at 4 points only)
    const int least = nf == tpt ? ppt : ppt - 1;      // points of the shortest thread
    const int RT = (s * d.h + least - 1) / least;
    if (least < d.h || RT > threads / 4) return w;    // at least half of the threads own points
    w.ppt = ppt;
    w.nw = nw;
    w.tpt = (int)tpt;
    w.nf = (int)nf;
    w.RT = RT;
    w.CT = (int)std::min<int64_t>(threads - 2 * RT, nth);
    w.NT = (int)((threads - 2) / tpt + 2);
    w.nblocks = (nth + w.CT - 1) / w.CT;
    w.lds = wave1d_lds_bytes(d.order, s, w.NT, d.L + d.m - 1, ppt, nw);
    w.ok = w.lds <= 64 * 1024;
    return w;
}

// Estimated time per step (us) of launches of s steps on region w.
// A step: one wave issues FP64 at nearly the rate of its SIMD and the oldest
// goes first, so a launch takes as long as the SIMD with the most waves: 0.035 +
// 0.0205 us per point of a thread for each of them, 6% more for ragged threads
// (the others have powers of two), but no less than one wave's latency; 0.01 us
// more for a wave with a tile face.  Measured at 1024 tiles of 1024 (us per
// step, points per thread x waves per SIMD), order 2: 16 x 2: 0.84, 8 x 3: 0.70,
// 20 x 1: 0.65, 10 x 2: 0.65; order 4: 8 x 3: 1.20, 12 x 2: 1.12, 20 x 1: 0.96.
// A launch: 3 us, the field's trip (1.7 us per 2^20 points, a seventh more where
// ragged threads make it unaligned), 0.2 us for each wave of a SIMD, 1.2 us for
// each history value a lane loads, 4 us where the field passes the stage in
// four parts.  Without that part the estimate took 20 to 32 points for few steps
// per launch on large grids (2^22 points, order 2, 2 steps: 24 points 10.0, 16:
// 7.9).  Over 1214 grids and step counts of 2^14 .. 2^24 points on tiles of 16 ..
// 4096 its choices take 1.5% more than the best kind, 3.9% without.
// stores: launches that write every fourth level from registers, coalesced only for
// few points per thread (2^20 points, order 2, us per step of a whole adjoint: 8
// points 3.66, 10 3.70, 20 3.84; order 4: 12 6.48, 20 6.59).
double fused_cost(const Derived &d, const FusedShape &w, int s, bool stores)
{
    const double nw = (double)w.nblocks * w.nw / 1024.0, waves = std::ceil(nw);
    const bool ragged = w.nf != w.tpt || (w.ppt & (w.ppt - 1)) != 0;
    const double mpts = (double)d.N / (1 << 20);
    const double hist = (double)(d.L + d.m - 1) * 2 * w.NT * d.h / (64.0 * w.nw);
    const double step = std::max(0.09 + 0.0215 * w.ppt,
                                 waves * (ragged ? 1.06 : 1.0) * (0.035 + 0.0205 * w.ppt));
    const double launch = 3.0 + 0.05 * w.ppt + (ragged ? 1.95 : 1.7) * mpts + 0.2 * nw +
                          1.2 * hist + (w.ppt >= 24 ? 4.0 : 0.0);
    return step * (d.order == 4 ? 1.5 : 1.0) * (d.contracted ? 0.8 : 1.0) +
           0.01 * waves * std::min(1.0, 64.0 / w.tpt) * d.h + launch / s +
           (stores ? (ragged ? 0.03 : 0.02) * w.ppt * mpts : 0.0);
}

// Grids on which variant 1 means the four-wave region (exact order: us per step
// with 2^24 points of order 4 in tiles of 4096, 48 steps: 8.86, one wave of 16: 9.87)
bool wide_grid(const Derived &d)
{
    return !d.contracted && d.N >= ((int64_t)1 << 23) && fused_shape(d, 32, kWide).ok;
}

// The kind of region of a fused launch of s steps: the one asked for where the
// tiles take it, else (0) the one of the least estimated time; 0 when no region
// fits this tile width.  Four-wave regions where a one-wave region would be rim by
// a quarter and more (order 4, 64 steps, us per step of four waves and of the best
// of one: 2^22 points in tiles of 4096 2.83 and 3.12, 2^24 9.10 and 9.60; 48 steps
// 2.94 and 2.71, 8.86 and 8.81).
int fused_kind(const Derived &d, int want, int s, bool stores = false)
{
    if (want != 0 && fused_shape(d, 1, want).ok) return want;
    if (!d.contracted && !stores && d.N >= ((int64_t)1 << 22) && s * d.h >= 112 &&
        fused_shape(d, s, kWide).ok)
        return kWide;
    int pick = 0;
    for (int t = s; pick == 0 && t >= 1; t /= 2) {           // (s may be more than any region takes)
        double least = 0.0;
        for (int p : kFusedKinds) {
            const FusedShape w = fused_shape(d, t, p);
            if (!w.ok) continue;
            const double cost = fused_cost(d, w, t, stores);
            if (pick == 0 || cost < least) { pick = p; least = cost; }
        }
    }
    return pick;
}

// Launches of at most f steps for the `left` ones, or one more where their
// number has to be odd (odd = 1) or even (0; < 0: any), so that the last of
// them writes the field the caller wants.  (Called again after each launch of
// ceil(left / launches) steps it counts down by one.)
int64_t launch_count(int64_t left, int64_t f, int odd)
{
    const int64_t n = (left + f - 1) / f;
    return odd >= 0 && (n & 1) != odd && n < left ? n + 1 : n;
}

// Steps the next launch advances when `left` remain and f are wanted per
// launch: as few launches as f, the region (which keeps at least half of its
// threads owned) and odd allow, of even length
int launch_steps(const Derived &d, int want, int f, int64_t left, int odd = -1)
{
    f = (int)std::min<int64_t>(f, left);
    const int kind = f > 1 ? fused_kind(d, want, f) : 0;
    while (kind && f > 1 && !fused_shape(d, f, kind).ok) --f;
    const int64_t n = launch_count(left, f, odd);
    return (int)((left + n - 1) / n);
}

// Points per thread of the whole-grid single-workgroup kernel (1D variant 4)
// for this context, 0 when the grid does not fit one workgroup
int whole_ppt(const at_ctx *c)
{
    const Derived &d = c->d;
    if (d.dim != 1) return 0;
    return step1d_whole_ppt(d.N, d.W, d.P, d.order, c->cfg.L + d.m - 1);
}

// Points per thread of the launches that rebuild every level of a checkpoint
// segment for single reverse steps: they write straight from registers,
// coalesced only for few points per thread
constexpr int kRebuildKind = 4;

// kind: the region asked for (fused_kind)
at_status launch_1d(at_ctx *c, const double *uin, double *uout, int64_t n0, int s, int publish,
                    int kind, double *levels = nullptr, int every = 1)
{
    const Derived &d = c->d;
    if (c->variant == kWholeVariant && !levels) {
        // the whole grid in one workgroup: any number of steps, no rims
        Step1D a{};
        a.uin = uin;
        a.uout = uout;
        a.ring = c->ring;
        a.delays = c->delays;
        a.N = d.N;
        a.P = d.P;
        a.W = d.W;
        a.n0 = n0;
        a.CH = d.N;
        a.s = s;
        a.R = c->lay.R;
        a.NT = (int)d.P;
        a.stale = c->cfg.halo_mode;
        a.publish = publish;
        a.RL = 0;
        a.slot0 = (int32_t)(n0 % a.R);
        a.D = c->cfg.L + d.m - 1;
        a.levels = nullptr;
        a.nu = c->cfg.nu;
        a.dt = c->cfg.dt;
        a.c1 = d.c1[0];
        a.c2 = d.c2[0];
        a.cadv = c->cfg.adv_speed;
        a.A1 = a.dt * a.c1;
        a.A2 = a.dt * (a.nu * a.c2);
        AT_HIP(launch_step1d_whole(a, d.order, c->cfg.adv_mode == 1, c->cfg.arith == 1,
                                   whole_ppt(c), c->st));
        return AT_OK;
    }
    // the fused kernels' regions, except for single steps of widths that the
    // one-step kernel takes and for the few widths the regions do not fit
    const int plain = s == 1 && !levels ? step1d_plain_ppt(d.W) : 0;
    const FusedShape ws = plain ? FusedShape() : fused_shape(d, s, fused_kind(d, kind, s));
    const Region1D rg = region_1d(d, s);
    const int reg = kThreads * rg.ppt;
    Step1D a{};
    a.uin = uin;
    a.uout = uout;
    a.ring = c->ring;
    a.delays = c->delays;
    a.N = d.N;
    a.P = d.P;
    a.W = d.W;
    a.n0 = n0;
    a.CH = rg.CH;
    if (a.CH < 1) return fail(AT_ERR_ARG, "fuse_steps %d too large for this stencil", s);
    a.s = s;
    a.R = c->lay.R;
    a.NT = (int)((reg - 1) / d.W + 2);
    a.stale = c->cfg.halo_mode;
    a.publish = publish;
    a.RL = (int32_t)rg.RL;
    a.slot0 = (int32_t)(n0 % a.R);
    a.D = c->cfg.L + d.m - 1;
    a.levels = levels;
    a.levels_every = every;
    if (levels && !ws.ok) return fail(AT_ERR_STATE, "level store needs the fused kernels");
    a.nu = c->cfg.nu;
    a.dt = c->cfg.dt;
    a.c1 = d.c1[0];
    a.c2 = d.c2[0];
    a.cadv = c->cfg.adv_speed;
    a.A1 = a.dt * a.c1;
    a.A2 = a.dt * (a.nu * a.c2);
    if (ws.ok) {
        a.tpt = ws.tpt;
        a.nf = ws.nf;
        a.CT = ws.CT;
        a.RT = ws.RT;
        a.NT = ws.NT;
        AT_HIP(launch_wave1d(a, d.order, c->cfg.adv_mode == 1, c->cfg.arith == 1, ws.ppt,
                             ws.nw, ws.nblocks, c->st));
        return AT_OK;
    }
    const int64_t nblocks = (d.N + a.CH - 1) / a.CH;
    AT_HIP(launch_step1d(a, d.order, c->cfg.adv_mode == 1, plain, c->cfg.arith == 1, nblocks,
                         c->st));
    return AT_OK;
}

}  // namespace

// 3D launcher (at_step3d.hip)
at_status at3_launch(at_ctx *c, const double *uin, double *uout, int64_t n0, int s, int publish);
at_status at3_publish(at_ctx *c, const double *u, int64_t n);
int at3_max_fuse(const at_ctx *c);
int at3_variants();
bool at3_variant_ok(const at_config *c, int var);
bool at3_is_aligned(int var);
bool at3_is_fused(int var);
int at3_single_variant(const at_config *c, int var);
int64_t at3_ws_capacity(const at_config *c);
at_status at3_launch_ws(at_ctx *ctx, double *u, double *scratch, int64_t n0, int64_t nsteps,
                        int32_t *cnt, int32_t *err, int8_t *delays, int32_t jitter, uint64_t seed,
                        int64_t spin_limit, int *in_scratch);

// accessors used by the 3D translation unit
extern "C++" {
const at_config *at_ctx_cfg(const at_ctx *c) { return &c->cfg; }
double *at_ctx_ring(const at_ctx *c) { return c->ring; }
const int8_t *at_ctx_delays(const at_ctx *c) { return c->delays; }
int at_ctx_R(const at_ctx *c) { return c->lay.R; }
hipStream_t at_ctx_stream(const at_ctx *c) { return c->st; }
void at_ctx_coefs(const at_ctx *c, double *c1, double *c2)
{
    for (int a = 0; a < 3; ++a) { c1[a] = c->d.c1[a]; c2[a] = c->d.c2[a]; }
}
at_status at_fail(at_status st, const char *msg) { return fail(st, "%s", msg); }
int at_ctx_variant(const at_ctx *c) { return c->variant; }
int32_t (*at_ctx_brick(at_ctx *c))[4] { return &c->brick; }
}

namespace {

at_status launch_any(at_ctx *c, const double *uin, double *uout, int64_t n0, int s, int publish,
                     int kind)
{
    if (c->d.dim == 1) return launch_1d(c, uin, uout, n0, s, publish, kind);
    return at3_launch(c, uin, uout, n0, s, publish);
}

// doubles in one field: N (1D) or (3 + nscalars) N (3D: velocity, then scalars)
int64_t field_doubles(const at_ctx *c)
{
    return (c->d.dim == 1 ? 1 : 3 + c->cfg.nscalars) * c->d.N;
}

int max_fuse(const at_ctx *c)
{
    return c->d.dim == 1 ? max_fuse_1d(c->d) : at3_max_fuse(c);
}

// Ring levels a later launch may still read once the context has reached
// level n1: 1D, the L + m - 1 levels below n1 (a step n reads levels down to
// n - L - m + 1 and publishes level n itself); 3D, levels n1 - L - 1 .. n1
// (a step reads levels down to n - L - 1, and level n's faces are published
// before it).  Levels below 0 are never read (start-up clamp).
void live_levels(const at_ctx *c, int64_t n1, int64_t *lo, int64_t *hi)
{
    if (c->d.dim == 1) {
        *lo = n1 - (c->cfg.L + c->d.m - 1);
        *hi = n1 - 1;
    } else {
        *lo = n1 - c->cfg.L - 1;
        *hi = n1;
    }
    if (*lo < 0) *lo = 0;
}

// The ring slots a context at step n may still read, from src to dst (two rings
// of this context's layout): the live levels, or in record mode every level so
// far.  A ring is sized for the most steps per launch and for the
// weakly-synchronous run, so the live slots are a small part of it (512^3, L = 3:
// one to five of ten levels of 302 MB; copying all ten took 1 ms).
hipError_t copy_ring(at_ctx *c, double *dst, const double *src, int64_t n)
{
    int64_t lo = 0, hi = n - 1;
    if (!c->cfg.record) live_levels(c, n, &lo, &hi);
    const int64_t R = c->lay.R, lev = (int64_t)ring_level_doubles(&c->cfg, c->d);
    hipError_t e = hipSuccess;
    while (e == hipSuccess && lo <= hi) {                 // contiguous slots, at most twice
        const int64_t slot = lo % R, count = std::min<int64_t>(hi - lo + 1, R - slot);
        e = launch_copy(dst + slot * lev, src + slot * lev, count * lev, c->st);
        lo += count;
    }
    return e;
}

// 1D variants.  0: by the estimate (fused_kind); 1, 2, 3: 16, 8, 4 points per
// thread in fused launches (1: the four-wave region on large grids)
int variant_points(int v) { return v == 0 ? 0 : (v == 1 ? 16 : (v == 2 ? 8 : 4)); }

int variant_kind(const Derived &d, int v)
{
    const int p = variant_points(v);
    return p == 16 && wide_grid(d) ? kWide : p;
}

void select_1d(at_ctx *c, int v)
{
    c->d.fppt = v ? variant_points(v) : fused_ppt(c->d);
    c->kind = variant_kind(c->d, v);
    c->variant = v;
}

// The region kind of every launch of a 1D run of nsteps steps: the variant's, or by
// the estimate at the steps per launch (so that variant and steps per launch name it)
int run_kind(const at_ctx *c, int64_t nsteps)
{
    if (c->d.dim != 1 || c->variant == kWholeVariant) return 0;
    int64_t s = std::max<int64_t>(1, std::min<int64_t>(c->fuse, nsteps));
    if (c->cfg.record) {                                  // (a segment's launches are even)
        const int64_t C = std::max<int64_t>(1, std::min<int64_t>(c->cfg.ckpt_every, nsteps));
        const int64_t launches = (C + s - 1) / s;
        s = (C + launches - 1) / launches;
    }
    return fused_kind(c->d, c->kind, (int)s);
}

// Steps of a run's next launch, `todo` before the end or the next checkpoint; home:
// the current level is in the caller's field
int64_t run_steps(const at_ctx *c, int kind, int64_t todo, bool home)
{
    if (c->d.dim != 1 || c->variant == kWholeVariant) return std::min<int64_t>(c->fuse, todo);
    // (one more launch, 7 us, instead of a copy back at the end where that takes
    // longer: 2^24 points 50 us)
    return launch_steps(c->d, kind, c->fuse, todo,
                        c->cfg.record || c->d.N < ((int64_t)1 << 21) ? -1 : (home ? 0 : 1));
}

// Debug mode AT_DEBUG_POISON_RING: after every launch, every ring slot that
// holds no live level is overwritten with NaN, so a step that read a level it
// must not would carry the NaN into the field.
hipError_t poison_ring(at_ctx *c, int64_t n1)
{
    if (!(c->debug & AT_DEBUG_POISON_RING)) return hipSuccess;
    int64_t lo, hi;
    live_levels(c, n1, &lo, &hi);
    const int64_t R = c->lay.R;
    const int64_t nlive = hi >= lo ? std::min<int64_t>(hi - lo + 1, R) : 0;
    return launch_poison(c->ring, R, (int64_t)ring_level_doubles(&c->cfg, c->d),
                         (int)(lo % R), (int)nlive, c->st);
}

// Clear the whole ring: zeros, or NaN in the poisoning debug mode (no level is
// live before the first step)
hipError_t clear_ring(at_ctx *c)
{
    const double v = (c->debug & AT_DEBUG_POISON_RING) ? __builtin_nan("") : 0.0;
    return launch_fill(c->ring, (int64_t)c->lay.R * (int64_t)ring_level_doubles(&c->cfg, c->d),
                       v, c->st);
}

void drop_graph(at_ctx *c)
{
    if (c->gexec) (void)hipGraphExecDestroy(c->gexec);
    c->gexec = nullptr;
    c->g_n0 = c->g_nsteps = -1;
}

// Steps of a tuning trial: whole launches of the candidate's s steps, an even
// number of them where the run allows it, compared per step (a run splits its
// steps evenly over its launches and prefers an even number, so a trial of the
// same length for all would make candidates alike)
int trial_length(int trial, int s, int64_t most)
{
    const int64_t n = ((int64_t)trial + s - 1) / s, pairs = (n + 1) / 2 * 2 * s;
    if (pairs <= most) return (int)pairs;
    return (int)(n * s <= most ? n * s : (trial >= s ? trial / s * s : trial));
}

// Points per thread that adj_fuse_max's regions are measured at (8 or 4: the
// larger one that still gives every SIMD four waves and divides the tile
// width), 0 when neither divides it
int adj_ppt(const Derived &d)
{
    if (d.W % 8 == 0 && d.N >= (int64_t)4 * 1024 * 64 * 8) return 8;
    if (d.W % 4 == 0) return 4;
    return d.W % 8 == 0 ? 8 : 0;
}

// Reverse steps per launch that at_set_adjoint_fuse accepts: 0 when the tiles
// do not fit the fused kernel, else the most (up to kMaxFuse) that keep the
// owned chunk of a 256-thread region at least half of it (and 256 points) and
// its LDS tables within 64 KiB.  (A launch takes as many of them as its own
// region allows, adj_shape.)
int adj_fuse_max(const Derived &d, int L)
{
    const int ppt = adj_ppt(d);
    if (ppt == 0) return 0;
    const int64_t reg = (int64_t)kThreads * ppt;
    int best = 0;
    for (int s = 1; s <= kMaxFuse; ++s) {
        const int64_t RL = ((int64_t)s * d.h + ppt - 1) / ppt * ppt;
        const int64_t CH = std::min<int64_t>((reg - RL - (int64_t)s * d.h) / ppt * ppt, d.N);
        if (CH < std::min<int64_t>(std::max<int64_t>(256, reg / 2), d.N)) break;
        const size_t lds = adj1d_fused_lds_bytes(d.order, s, (int)((reg - 1) / d.W + 2), L) +
                           8 * (size_t)8 * d.h * kThreads;
        if (lds > 64 * 1024) break;
        best = s;
    }
    return best;
}

// The region of the fused reverse launches of S steps (a multiple of
// kAdjGroup): one wave, rims of (S + kAdjGroup) h points, LDS tables within
// 64 KiB; S = 0: none.
struct RegionAdj {
    int S = 0, ppt = 0, NT = 0, tpt = 0, nf = 0, CT = 0, RT = 0;
    int64_t nblocks = 0;
};

RegionAdj adj_shape(const Derived &d, int L, int ppt, int s)
{
    RegionAdj r;
    const int64_t tpt = (d.W + ppt - 1) / ppt, nf = d.W - tpt * (ppt - 1), nth = d.P * tpt;
    if (nf < 1 || d.W > ((int64_t)1 << 30) || nth >= ((int64_t)1 << 31) - 256) return r;
    if (nf == tpt && ppt != 8 && ppt != 4) return r;          // (built for ragged tiles only)
    const int least = nf == tpt ? ppt : ppt - 1;
    r.RT = ((s + kAdjGroup) * d.h + least - 1) / least;
    r.NT = (int)(62 / tpt + 2);
    if (r.RT > 16 || adj1d_fused_lds_bytes(d.order, s, r.NT, L) > 64 * 1024) return r;
    r.S = s;
    r.ppt = ppt;
    r.tpt = (int)tpt;
    r.nf = (int)nf;
    r.CT = (int)std::min<int64_t>(64 - 2 * r.RT, nth);
    r.nblocks = (nth + r.CT - 1) / r.CT;
    return r;
}

// The points per thread and the most steps per launch of a sweep over segments
// of at most `seg` steps, by an estimate of the time per step.  One wave issues
// FP64 at nearly the rate of its SIMD and the oldest goes first, so a launch
// takes as long as the SIMD with the most waves: 0.3 + 0.093 us per point of a
// lane for each of them and step, and 7 us before the first.  (2^20 points,
// order 2, us per step, waves per SIMD: 10 and 9 points 2.9 with 2, 8 points 3.4
// with 2.4, 4 points 3.7 with 4.9.)
RegionAdj adj_region(const Derived &d, int L, int64_t seg)
{
    RegionAdj best;
    double least = 0.0;
    for (int ppt : {10, 8, 6, 4})
        for (int s = kAdjGroup; s <= kMaxFuse; s += kAdjGroup) {
            const RegionAdj r = adj_shape(d, L, ppt, s);
            if (r.S == 0) break;
            const int64_t wgs = 160 * 1024 / (int64_t)adj1d_fused_lds_bytes(d.order, s, r.NT, L);
            const int64_t at_once = 256 * std::min<int64_t>(wgs, 4);
            const int64_t launches = (seg + s - 1) / s;
            const double t = (double)((r.nblocks + at_once - 1) / at_once) * (0.3 + 0.093 * ppt) +
                             7.0 * (double)launches / (double)seg;
            if (best.S == 0 || t < least) { best = r; least = t; }
        }
    return best;
}

}  // namespace

extern "C" {

int32_t at_abi_version(void) { return AT_ABI_VERSION; }

const char *at_last_error(void) { return g_err.c_str(); }

uint64_t at_config_bytes(void) { return sizeof(at_config); }

at_status at_workspace_bytes(const at_config *cfg, uint64_t *bytes)
{
    Derived d;
    at_status st = derive(cfg, d);
    if (st) return st;
    if (!bytes) return fail(AT_ERR_ARG, "null output");
    Layout L;
    make_layout(cfg, d, L);
    *bytes = L.total;
    return AT_OK;
}

at_status at_init(const at_config *cfg, at_ctx **out)
{
    if (!out) return fail(AT_ERR_ARG, "null output");
    *out = nullptr;
    Derived d;
    at_status st = derive(cfg, d);
    if (st) return st;
    Layout L;
    make_layout(cfg, d, L);
    if (!cfg->workspace) return fail(AT_ERR_ARG, "workspace is NULL");
    if (((uintptr_t)cfg->workspace) % kAlign) return fail(AT_ERR_ARG, "workspace not 256-byte aligned");
    if (cfg->workspace_bytes < L.total)
        return fail(AT_ERR_NOMEM, "workspace %llu bytes, need %llu",
                    (unsigned long long)cfg->workspace_bytes, (unsigned long long)L.total);
    if (cfg->delay_mode == AT_DELAY_HOST) {
        // every entry must satisfy 0 <= k <= min(L, max(0, n - m + 1))
        for (int64_t n = 0; n < cfg->nsteps_max; ++n) {
            int64_t lim = std::min<int64_t>(cfg->L, std::max<int64_t>(0, n - d.m + 1));
            const int8_t *row = cfg->delays_host + n * d.F;
            for (int64_t f = 0; f < d.F; ++f)
                if (row[f] < 0 || row[f] > lim)
                    return fail(AT_ERR_DELAY, "delay k[%lld][%lld] = %d outside 0..%lld",
                                (long long)n, (long long)f, (int)row[f], (long long)lim);
        }
    }
    at_ctx *c = new (std::nothrow) at_ctx;
    if (!c) return fail(AT_ERR_NOMEM, "host allocation failed");
    c->cfg = *cfg;
    c->cfg.delays_host = nullptr;
    c->d = d;
    c->lay = L;
    c->st = (hipStream_t)cfg->stream;
    char *base = (char *)cfg->workspace;
    c->delays = (int8_t *)(base + L.delays);
    c->ring = (double *)(base + L.ring);
    c->red = (double *)(base + L.red);
    c->sync = (int32_t *)(base + L.sync);
    c->ckpt = cfg->record ? (double *)(base + L.ckpt) : nullptr;
    c->seg = cfg->record ? (double *)(base + L.seg) : nullptr;
    c->lam = cfg->record ? (double *)(base + L.lam) : nullptr;
    c->mu = cfg->record ? (double *)(base + L.mu) : nullptr;
    c->gnu = cfg->record ? (double *)(base + L.gnu) : nullptr;
    c->n = 0;
    c->variant = 0;
    if (d.dim == 3)   // the first variant with a build for this component count
        while (!at3_variant_ok(&c->cfg, c->variant)) ++c->variant;
    c->fuse = cfg->fuse_steps > 0 ? std::min(cfg->fuse_steps, max_fuse(c)) : 1;
    if (d.dim == 3 && c->fuse == 2)   // two steps per launch: the two-step kernel
        c->variant = at3_variant_ok(&c->cfg, 15) ? 15 : 16;
    hipError_t e = hipSuccess;
    if (cfg->delay_mode == AT_DELAY_GENERATE)
        e = launch_delays(c->delays, cfg->nsteps_max, d.F, cfg->L, d.m, cfg->delay_dist,
                          cfg->delay_seed, c->st);
    else if (cfg->nsteps_max > 0)
        e = hipMemcpyAsync(c->delays, cfg->delays_host, (size_t)(cfg->nsteps_max * d.F),
                           hipMemcpyHostToDevice, c->st);
    if (e == hipSuccess)
        e = launch_fill(c->ring, (int64_t)L.R * (int64_t)ring_level_doubles(cfg, d), 0.0, c->st);
    if (e == hipSuccess) e = hipStreamSynchronize(c->st);
    if (e != hipSuccess) {
        delete c;
        return fail(AT_ERR_HIP, "at_init: %s", hipGetErrorString(e));
    }
    *out = c;
    return AT_OK;
}

void at_free(at_ctx *c)
{
    if (!c) return;
    drop_graph(c);
    if (c->cap) (void)hipStreamDestroy(c->cap);
    delete c;
}

at_status at_set_graph(at_ctx *c, int32_t use_graph)
{
    if (!c) return fail(AT_ERR_ARG, "null context");
    if (use_graph != 0 && use_graph != 1) return fail(AT_ERR_ARG, "use_graph must be 0 or 1");
    c->use_graph = use_graph;
    if (!use_graph) drop_graph(c);
    return AT_OK;
}

at_status at_set_debug(at_ctx *c, int32_t flags)
{
    if (!c) return fail(AT_ERR_ARG, "null context");
    if (flags & ~AT_DEBUG_POISON_RING) return fail(AT_ERR_ARG, "unknown debug flags 0x%x", flags);
    if ((flags & AT_DEBUG_POISON_RING) && c->cfg.record)
        return fail(AT_ERR_STATE, "ring poisoning is not available in record mode (the adjoint "
                                  "re-reads every level)");
    const bool was = c->debug & AT_DEBUG_POISON_RING;
    c->debug = flags;
    if ((flags & AT_DEBUG_POISON_RING) && !was) {
        if (c->n == 0) AT_HIP(clear_ring(c));
        else AT_HIP(poison_ring(c, c->n));
    }
    return AT_OK;
}

at_status at_set_fuse(at_ctx *c, int32_t s)
{
    if (!c) return fail(AT_ERR_ARG, "null context");
    if (s < 1 || s > kMaxFuse) return fail(AT_ERR_ARG, "fuse_steps must be in 1..%d", kMaxFuse);
    const int mf = max_fuse(c);
    if (s > mf) return fail(AT_ERR_ARG, "fuse_steps %d exceeds the limit %d of this grid", s, mf);
    c->fuse = s;
    if (c->d.dim == 3) {   // 3D: the kernel variant follows the steps per launch
        if (s == 2 && !at3_is_fused(c->variant))
            c->variant = at3_variant_ok(&c->cfg, 15) ? 15 : 16;
        if (s == 1) c->variant = at3_single_variant(&c->cfg, c->variant);
    }
    return AT_OK;
}

at_status at_set_adjoint_fuse(at_ctx *c, int32_t s)
{
    if (!c) return fail(AT_ERR_ARG, "null context");
    if (s < 0 || s > kMaxFuse) return fail(AT_ERR_ARG, "adjoint steps per launch must be in 0..%d",
                                           kMaxFuse);
    if (s > 1) {
        if (c->d.dim != 1) return fail(AT_ERR_ARG, "the adjoint is 1D only");
        const int mf = adj_fuse_max(c->d, c->cfg.L);
        if (s > mf)
            return fail(AT_ERR_ARG, "%d reverse steps per launch exceed the limit %d of this grid",
                        s, mf);
    }
    c->adj_fuse = s;
    return AT_OK;
}

at_status at_set_variant(at_ctx *c, int32_t v)
{
    if (!c) return fail(AT_ERR_ARG, "null context");
    const int nv = c->d.dim == 1 ? 5 : at3_variants();
    if (v < 0 || v >= nv) return fail(AT_ERR_ARG, "variant must be in 0..%d", nv - 1);
    if (c->d.dim == 3 && !at3_variant_ok(&c->cfg, v))
        return fail(AT_ERR_ARG, "variant %d needs block widths that are multiples of its tile", v);
    if (c->d.dim == 1 && v == kWholeVariant) {
        if (whole_ppt(c) == 0)
            return fail(AT_ERR_ARG, "variant 4 needs the grid in one workgroup (N <= 256 x 16, "
                                    "N and the tile width multiples of 4)");
        c->variant = v;
        c->fuse = (int)std::min<int64_t>(std::max<int64_t>(c->cfg.nsteps_max, 1), INT32_MAX);
        return AT_OK;
    }
    if (c->d.dim == 1) {
        const int p = variant_points(v);
        if (p && c->d.W % p != 0)
            return fail(AT_ERR_ARG, "variant %d needs a tile width divisible by %d", v, p);
        select_1d(c, v);
        c->fuse = std::min(c->fuse, max_fuse(c));
    } else {
        c->fuse = at3_is_fused(v) ? 2 : 1;   // 3D: two-step variants advance two steps per launch
    }
    c->variant = v;
    return AT_OK;
}

at_status at_query(const at_ctx *c, int64_t *n, int32_t *fuse, int32_t *R, int32_t *variant)
{
    if (!c) return fail(AT_ERR_ARG, "null context");
    if (n) *n = c->n;
    if (fuse) *fuse = c->fuse;
    if (R) *R = c->lay.R;
    if (variant) *variant = c->variant;
    return AT_OK;
}

at_status at_launch_shape(const at_ctx *c, int64_t nsteps, int32_t *steps, int32_t *points,
                          int32_t *waves)
{
    if (!c) return fail(AT_ERR_ARG, "null context");
    if (c->d.dim != 1) return fail(AT_ERR_ARG, "the launch shape is a 1D context's");
    if (nsteps < 1) return fail(AT_ERR_ARG, "nsteps < 1");
    const int64_t C = c->cfg.ckpt_every;
    const int64_t todo = c->cfg.record ? std::min<int64_t>(nsteps, C - c->n % C) : nsteps;
    const int kind = run_kind(c, nsteps);
    const int s = (int)run_steps(c, kind, todo, true);
    const int plain = s == 1 ? step1d_plain_ppt(c->d.W) : 0;
    const FusedShape w = plain ? FusedShape() : fused_shape(c->d, s, fused_kind(c->d, kind, s));
    const bool whole = c->variant == kWholeVariant;
    if (steps) *steps = s;
    if (points) *points = whole ? whole_ppt(c) : (w.ok ? w.ppt : (plain ? plain : step1d_points_per_thread()));
    if (waves) *waves = !whole && w.ok ? w.nw : kThreads / 64;
    return AT_OK;
}

at_status at_step(at_ctx *c, const double *u_in, double *u_out)
{
    if (!c || !u_in || !u_out) return fail(AT_ERR_ARG, "null argument");
    if (u_in == u_out) return fail(AT_ERR_ARG, "u_in and u_out must differ");
    if (c->n + 1 > c->cfg.nsteps_max) return fail(AT_ERR_STATE, "step %lld beyond nsteps_max",
                                                  (long long)c->n);
    if (c->cfg.record && c->n % c->cfg.ckpt_every == 0)
        AT_HIP(launch_copy(c->ckpt + (c->n / c->cfg.ckpt_every) * c->d.N, u_in, c->d.N, c->st));
    if (c->d.dim == 3) {                      // the face values of level n, from u_in
        const at_status sp = at3_publish(c, u_in, c->n);
        if (sp) return sp;
    }
    at_status st = launch_any(c, u_in, u_out, c->n, 1, 1, c->kind);
    if (st) return st;
    c->n += 1;
    AT_HIP(poison_ring(c, c->n));
    return AT_OK;
}

namespace {

// the launch sequence of at_run on c->st (recorded into a graph when c->st is
// a capturing stream); advances c->n
at_status run_launches(at_ctx *c, double *u, double *scratch, int64_t nsteps)
{
    double *cur = u, *oth = scratch;
    int64_t left = nsteps;
    const int64_t C = c->cfg.ckpt_every;
    const int kind = run_kind(c, nsteps);
    if (c->d.dim == 3 && nsteps > 0) {        // the face values of level n, from u
        const at_status sp = at3_publish(c, u, c->n);
        if (sp) return sp;
    }
    while (left > 0) {
        int64_t todo = left;                  // steps up to the next checkpoint or the end
        if (c->cfg.record) {
            if (c->n % C == 0)
                AT_HIP(launch_copy(c->ckpt + (c->n / C) * c->d.N, cur, c->d.N, c->st));
            todo = std::min<int64_t>(todo, C - c->n % C);
        }
        const int64_t s = run_steps(c, kind, todo, cur == u);
        // 1D without the edge tape: only the last L + m - 1 levels of a launch
        // reach the ring (the next launch reads no older level)
        at_status st = launch_any(c, cur, oth, c->n, (int)s,
                                  (c->d.dim == 1 && !c->cfg.record) ? 2 : 1, kind);
        if (st) return st;
        std::swap(cur, oth);
        c->n += s;
        left -= s;
        AT_HIP(poison_ring(c, c->n));
    }
    if (cur != u) AT_HIP(launch_copy(u, cur, field_doubles(c), c->st));
    return AT_OK;
}

}  // namespace

at_status at_run(at_ctx *c, double *u, double *scratch, int64_t nsteps)
{
    if (!c || !u || !scratch) return fail(AT_ERR_ARG, "null argument");
    if (u == scratch) return fail(AT_ERR_ARG, "u and scratch must differ");
    if (nsteps < 0) return fail(AT_ERR_ARG, "nsteps < 0");
    if (c->n + nsteps > c->cfg.nsteps_max)
        return fail(AT_ERR_STATE, "run to step %lld beyond nsteps_max %lld",
                    (long long)(c->n + nsteps), (long long)c->cfg.nsteps_max);
    if (!c->use_graph || nsteps == 0) return run_launches(c, u, scratch, nsteps);
    // graph replay: the cached graph applies when it was captured for the same
    // start step, length, fields and launch choices (a 1D region kind follows from
    // variant, steps per launch and length)
    if (!(c->gexec && c->g_n0 == c->n && c->g_nsteps == nsteps && c->g_u == u &&
          c->g_s == scratch && c->g_fuse == c->fuse && c->g_variant == c->variant &&
          c->g_debug == c->debug)) {
        drop_graph(c);
        if (!c->cap) AT_HIP(hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking));
        const int64_t n0 = c->n;
        hipStream_t own = c->st;
        c->st = c->cap;
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamBeginCapture(c->cap, hipStreamCaptureModeThreadLocal);
        at_status st = AT_OK;
        if (e == hipSuccess) {
            st = run_launches(c, u, scratch, nsteps);
            hipError_t e2 = hipStreamEndCapture(c->cap, &g);
            if (e2 != hipSuccess && st == AT_OK) e = e2;
        }
        c->st = own;
        c->n = n0;
        if (st) {
            if (g) (void)hipGraphDestroy(g);
            return st;
        }
        if (e != hipSuccess) return fail(AT_ERR_HIP, "graph capture: %s", hipGetErrorString(e));
        e = hipGraphInstantiate(&c->gexec, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) {
            c->gexec = nullptr;
            return fail(AT_ERR_HIP, "graph instantiate: %s", hipGetErrorString(e));
        }
        c->g_n0 = n0;
        c->g_nsteps = nsteps;
        c->g_u = u;
        c->g_s = scratch;
        c->g_fuse = c->fuse;
        c->g_variant = c->variant;
        c->g_debug = c->debug;
    }
    AT_HIP(hipGraphLaunch(c->gexec, c->st));
    c->n += nsteps;
    return AT_OK;
}

at_status at_ws_capacity(const at_ctx *c, int64_t *max_tiles)
{
    if (!c || !max_tiles) return fail(AT_ERR_ARG, "null argument");
    *max_tiles = 0;
    if (c->d.dim == 3) {
        *max_tiles = at3_ws_capacity(&c->cfg);
        return AT_OK;
    }
    *max_tiles = ws1d_max_tiles(c->d.order, c->cfg.adv_mode == 1, c->d.W);
    return AT_OK;
}

at_status at_run_ws(at_ctx *c, double *u, double *scratch, int64_t nsteps, int32_t jitter,
                    uint64_t seed, int64_t spin_limit)
{
    if (!c || !u) return fail(AT_ERR_ARG, "null argument");
    if (c->cfg.record) return fail(AT_ERR_STATE, "the weakly-synchronous run has no record mode");
    if (c->cfg.arith != 0) return fail(AT_ERR_ARG, "the weakly-synchronous run uses arith 0");
    if (c->n != 0) return fail(AT_ERR_STATE, "the weakly-synchronous run starts at step 0");
    if (nsteps < 0 || nsteps > c->cfg.nsteps_max)
        return fail(AT_ERR_ARG, "nsteps must be in 0..nsteps_max");
    if (nsteps >= ((int64_t)1 << 31) - 1) return fail(AT_ERR_ARG, "nsteps too large");
    if (jitter < 0 || jitter > (1 << 20)) return fail(AT_ERR_ARG, "jitter must be in 0..2^20");
    const Derived &d = c->d;
    const int64_t spins = spin_limit > 0 ? spin_limit : ((int64_t)1 << 20);
    if (d.dim == 3) {
        if (!scratch || scratch == u)
            return fail(AT_ERR_ARG, "the 3D weakly-synchronous run needs a scratch field apart from u");
        const int64_t Wx = c->cfg.n[0] / c->cfg.p[0], Wy = c->cfg.n[1] / c->cfg.p[1];
        if (Wx % 64 != 0 || Wy % 8 != 0)
            return fail(AT_ERR_SHAPE, "3D weakly-synchronous run: block widths must be multiples "
                                      "of 64 (x) and 8 (y)");
        const int64_t maxb = at3_ws_capacity(&c->cfg);
        if (d.nb > maxb)
            return fail(AT_ERR_SHAPE, "%lld blocks, but at most %lld workgroups can be resident "
                                      "at once", (long long)d.nb, (long long)maxb);
        if (nsteps == 0) return AT_OK;
        int32_t *err = c->sync + d.nb;
        const at_status sp = at3_publish(c, u, 0);           // level 0's faces, announced below
        if (sp) return sp;
        AT_HIP(launch_ws_init(c->sync, d.nb, 0, err, c->st));
        int in_scratch = 0;
        const at_status st = at3_launch_ws(c, u, scratch, 0, nsteps, c->sync, err, c->delays,
                                           jitter, seed, spins, &in_scratch);
        if (st) return st;
        if (in_scratch) AT_HIP(launch_copy(u, scratch, field_doubles(c), c->st));
        int32_t herr = 0;
        AT_HIP(hipMemcpyAsync(&herr, err, sizeof herr, hipMemcpyDeviceToHost, c->st));
        AT_HIP(hipStreamSynchronize(c->st));
        if (herr != 0)
            return fail(AT_ERR_TIMEOUT, "a wait passed the spin limit; u and the delays are undefined");
        c->n = nsteps;
        return AT_OK;
    }
    int nt = 0, ppt = 0;
    if (!ws1d_shape(d.W, d.h, &nt, &ppt))
        return fail(AT_ERR_SHAPE, "tile width must be 256 q or 64 q with q in {1, 2, 4, 8, 16} "
                                  "(q >= 2 for order 4)");
    const bool linear = c->cfg.adv_mode == 1;
    const int64_t maxt = ws1d_max_tiles(d.order, linear, d.W);
    if (d.P > maxt)
        return fail(AT_ERR_SHAPE, "%lld tiles, but at most %lld workgroups can be resident at once",
                    (long long)d.P, (long long)maxt);
    if (nsteps == 0) return AT_OK;
    int32_t *err = c->sync;
    Ws1D a{};
    a.u = u;
    a.ring = c->ring;
    a.err = err;
    a.delays = c->delays;
    a.P = d.P;
    a.W = d.W;
    a.n0 = 0;
    a.nsteps = nsteps;
    a.spin_limit = spins;
    a.R = c->lay.R;
    a.L = c->cfg.L;
    a.stale = c->cfg.halo_mode;
    a.jitter = jitter;
    a.seed = seed;
    a.coef.nu = c->cfg.nu;
    a.coef.dt = c->cfg.dt;
    a.coef.c1 = d.c1[0];
    a.coef.c2 = d.c2[0];
    a.coef.cadv = c->cfg.adv_speed;
    AT_HIP(launch_ws1d(a, d.order, linear, c->st));
    int32_t herr = 0;
    AT_HIP(hipMemcpyAsync(&herr, err, sizeof herr, hipMemcpyDeviceToHost, c->st));
    AT_HIP(hipStreamSynchronize(c->st));
    if (herr != 0)
        return fail(AT_ERR_TIMEOUT, "a wait passed the spin limit; u and the delays are undefined");
    c->n = nsteps;
    return AT_OK;
}

at_status at_autotune(at_ctx *c, const double *u0, double *t1, double *t2, int32_t trial_steps,
                      int32_t *chosen)
{
    if (!c || !u0 || !t1 || !t2) return fail(AT_ERR_ARG, "null argument");
    if (c->n != 0) return fail(AT_ERR_STATE, "autotune needs a context at step 0");
    if (c->cfg.record) return fail(AT_ERR_STATE, "autotune is not available in record mode");
    if (trial_steps < 1 || trial_steps > c->cfg.nsteps_max)
        return fail(AT_ERR_ARG, "trial_steps must be in 1..nsteps_max");
    // (variant, steps per launch) pairs as at_set_variant and at_set_fuse take them
    std::vector<std::pair<int, int>> cands;
    if (c->d.dim == 1) {
        // of each region kind that a variant names (0: the estimate's at that many
        // steps) the most steps for each number of waves per SIMD, and a few round
        // counts; of those the twelve of the least estimates
        std::vector<std::pair<double, std::pair<int, int>>> est;
        for (int v : {1, 2, 3, 0}) {
            Derived d = c->d;
            if (v && d.W % variant_points(v) != 0) continue;
            d.fppt = v ? variant_points(v) : fused_ppt(d);
            const int mf = max_fuse_1d(d);
            int64_t waves = 0;
            int last = 0;
            for (int s = std::min(mf, kMaxFuse); s >= 2; --s) {
                const int kind = v ? variant_kind(d, v) : fused_kind(d, 0, s);
                bool named = false;                      // by one of the variants above
                for (int w = 1; w <= 3; ++w)
                    named = named || (v == 0 && d.W % variant_points(w) == 0 && variant_kind(d, w) == kind);
                const FusedShape w = fused_shape(d, s, kind);
                if (!w.ok || named) continue;
                const int64_t now = (w.nblocks * w.nw + 1023) / 1024;
                if (kind == last && now == waves && s % 16 != 0 && (s > 16 || s % 4 != 0)) continue;
                waves = now;
                last = kind;
                // (always tried on the large grids)
                if (kind == kWide && v == 1 && (s == 32 || s == 40 || s == 48 || s == 64))
                    cands.push_back({v, s});
                else if (kind != kWide) est.push_back({fused_cost(d, w, s, false), {v, s}});
            }
        }
        std::sort(est.begin(), est.end());
        for (size_t i = 0; i < est.size() && i < 12; ++i) cands.push_back(est[i].second);
        if (cands.empty()) {                                  // widths without such regions
            const int mf = max_fuse(c);
            for (int s : {64, 32, 16, 8, 4})
                if (s <= mf) cands.push_back({0, s});
            cands.push_back({0, 1});
        }
        if (whole_ppt(c) != 0) cands.push_back({kWholeVariant, 0});   // one launch per run
    } else {
        for (int v = 0; v < at3_variants(); ++v)
            if (at3_variant_ok(&c->cfg, v) && (at3_is_aligned(v) || at3_is_fused(v) || cands.empty() || v == 9))
                cands.push_back({v, at3_is_fused(v) ? 2 : 1});   // (the others are one of two kernels)
    }
    hipEvent_t e0, e1;
    AT_HIP(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(AT_ERR_HIP, "at_autotune: hipEventCreate failed");
    }
    std::vector<float> ms_best(cands.size(), 1e30f);
    const int keep_graph = c->use_graph;
    c->use_graph = 0;                         // time the launches themselves
    at_status st = AT_OK;
    // select a candidate
    auto choose = [&](std::pair<int, int> vs) {
        c->variant = vs.first;
        c->fuse = vs.second;
        if (c->d.dim != 1) return;
        select_1d(c, vs.first == kWholeVariant ? 0 : vs.first);
        if (vs.first == kWholeVariant) {
            c->variant = kWholeVariant;
            c->fuse = (int)std::min<int64_t>(c->cfg.nsteps_max, INT32_MAX);
        }
    };
    // twice over all candidates, not twice each: an idle device's clock takes some
    // ten milliseconds to rise, and the first trials pay for it (2^24 points: 12.1
    // us per step, later 9.3); then twice more over those within 5% of the best
    for (int rep = 0; rep < 4; ++rep) {
        const float near = 1.05f * *std::min_element(ms_best.begin(), ms_best.end());
        for (size_t i = 0; i < cands.size() && st == AT_OK; ++i) {
            if (rep >= 2 && ms_best[i] > near) continue;
            choose(cands[i]);
            // (a run of the whole-grid variant is one launch, whatever its length)
            const int s = c->d.dim == 1 && c->variant == kWholeVariant ? kMaxFuse : c->fuse;
            const int steps = trial_length(trial_steps, s, c->cfg.nsteps_max);
            hipError_t e = clear_ring(c);
            if (e == hipSuccess) e = launch_copy(t1, u0, field_doubles(c), c->st);
            c->n = 0;
            if (e == hipSuccess) e = hipEventRecord(e0, c->st);
            if (e == hipSuccess) st = at_run(c, t1, t2, steps);
            if (e == hipSuccess && st == AT_OK) e = hipEventRecord(e1, c->st);
            if (e == hipSuccess && st == AT_OK) e = hipEventSynchronize(e1);
            float ms = 0.f;
            if (e == hipSuccess && st == AT_OK) e = hipEventElapsedTime(&ms, e0, e1);
            if (e != hipSuccess && st == AT_OK)
                st = fail(AT_ERR_HIP, "at_autotune: %s", hipGetErrorString(e));
            ms_best[i] = std::min(ms_best[i], ms / (float)steps);
        }
    }
    // the candidates expected to be best come first: another has to be 1% faster
    size_t pick = 0;
    for (size_t i = 1; i < cands.size(); ++i)
        if (ms_best[i] < ms_best[pick] * 0.99f) pick = i;
    const std::pair<int, int> best = cands[pick];
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    c->use_graph = keep_graph;
    c->n = 0;
    if (st) return st;
    choose(best);
    AT_HIP(clear_ring(c));
    AT_HIP(hipStreamSynchronize(c->st));
    if (chosen) *chosen = c->d.dim == 1 ? c->fuse : best.first;
    return AT_OK;
}

at_status at_delays_copy(const at_ctx *c, int8_t *host_out)
{
    if (!c || !host_out) return fail(AT_ERR_ARG, "null argument");
    AT_HIP(hipMemcpyAsync(host_out, c->delays, (size_t)(c->cfg.nsteps_max * c->d.F),
                          hipMemcpyDeviceToHost, c->st));
    AT_HIP(hipStreamSynchronize(c->st));
    return AT_OK;
}

at_status at_snapshot_bytes(const at_ctx *c, uint64_t *bytes)
{
    if (!c || !bytes) return fail(AT_ERR_ARG, "null argument");
    *bytes = align_up(8ull * field_doubles(c)) +
             align_up(8ull * c->lay.R * ring_level_doubles(&c->cfg, c->d)) + kAlign;
    return AT_OK;
}

at_status at_snapshot(at_ctx *c, const double *u, void *dev_buf)
{
    if (!c || !u || !dev_buf) return fail(AT_ERR_ARG, "null argument");
    const uint64_t nu = field_doubles(c), nr = (uint64_t)c->lay.R * ring_level_doubles(&c->cfg, c->d);
    char *b = (char *)dev_buf;
    AT_HIP(launch_copy((double *)b, u, nu, c->st));
    if (c->debug & AT_DEBUG_POISON_RING)                  // the poison too
        AT_HIP(launch_copy((double *)(b + align_up(8 * nu)), c->ring, nr, c->st));
    else
        AT_HIP(copy_ring(c, (double *)(b + align_up(8 * nu)), c->ring, c->n));
    // the step counter, exact below 2^53, written by a kernel (no host buffer
    // has to outlive the call, so nothing waits)
    AT_HIP(launch_fill((double *)(b + align_up(8 * nu) + align_up(8 * nr)), 1, (double)c->n,
                       c->st));
    for (auto &e : c->snaps)
        if (e.first == dev_buf) { e.second = c->n; return AT_OK; }
    c->snaps.emplace_back(dev_buf, c->n);
    return AT_OK;
}

at_status at_restore(at_ctx *c, const void *dev_buf, double *u)
{
    if (!c || !u || !dev_buf) return fail(AT_ERR_ARG, "null argument");
    const uint64_t nu = field_doubles(c), nr = (uint64_t)c->lay.R * ring_level_doubles(&c->cfg, c->d);
    const char *b = (const char *)dev_buf;
    // a buffer this context filled: its step is known on the host; any other
    // buffer: read the step it holds (the only case that waits for the stream)
    int64_t step = -1;
    for (const auto &e : c->snaps)
        if (e.first == dev_buf) step = e.second;
    if (step < 0) {
        double nn = 0.0;
        AT_HIP(hipMemcpyAsync(&nn, b + align_up(8 * nu) + align_up(8 * nr), sizeof nn,
                              hipMemcpyDeviceToHost, c->st));
        AT_HIP(hipStreamSynchronize(c->st));
        if (!(nn >= 0.0) || nn > (double)c->cfg.nsteps_max || nn != floor(nn))
            return fail(AT_ERR_ARG, "buffer does not hold a snapshot of this context");
        step = (int64_t)nn;
    }
    AT_HIP(launch_copy(u, (const double *)b, nu, c->st));
    AT_HIP(copy_ring(c, c->ring, (const double *)(b + align_up(8 * nu)), step));
    c->n = step;
    AT_HIP(poison_ring(c, step));                         // debug mode: the other slots
    return AT_OK;
}

at_status at_stats(at_ctx *c, const double *u, double *out4)
{
    if (!c || !u || !out4) return fail(AT_ERR_ARG, "null argument");
    const int64_t n = field_doubles(c);
    AT_HIP(launch_stats(u, n, c->red, out4, c->st));
    return AT_OK;
}

at_status at_loss(at_ctx *c, const double *u, const double *target, double *lam, double *J_dev)
{
    if (!c || !u || !target || !J_dev) return fail(AT_ERR_ARG, "null argument");
    const int64_t n = field_doubles(c);
    AT_HIP(launch_loss(u, target, lam, n, c->red, J_dev, c->st));
    return AT_OK;
}

at_status at_adjoint(at_ctx *c, const double *lambda_T, double *grad_u0, double *grad_nu_dev)
{
    if (!c || !lambda_T || !grad_u0 || !grad_nu_dev) return fail(AT_ERR_ARG, "null argument");
    if (!c->cfg.record) return fail(AT_ERR_STATE, "at_adjoint needs a context in record mode");
    const Derived &d = c->d;
    const int64_t nend = c->n, C = c->cfg.ckpt_every, N = d.N;
    double *lcur = c->lam, *loth = c->lam + N;
    const RegionAdj rg = adj_region(d, c->cfg.L, std::max<int64_t>(1, std::min(C, nend)));
    AT_HIP(launch_copy(lcur, lambda_T, N, c->st));
    AT_HIP(launch_fill(c->mu, (int64_t)c->lay.Rmu * d.P * 2 * d.h, 0.0, c->st));
    AT_HIP(launch_fill(c->gnu, 2 * c->lay.ngnu, 0.0, c->st));
    if (nend > 0) {
        for (int64_t a0 = ((nend - 1) / C) * C; a0 >= 0; a0 -= C) {
            const int64_t a1 = std::min(a0 + C, nend);
            AT_HIP(launch_copy(c->seg, c->ckpt + (a0 / C) * N, N, c->st));
            // rebuild the levels the reverse launches read, every kAdjGroup-th of
            // a0 .. a1-1 (each for single reverse steps): fused launches that store
            // them on the way, or one launch per step for the tile widths the
            // fused kernels do not take
            const int smax = rg.S;
            const int sadj = c->adj_fuse == 0 ? smax : (c->adj_fuse == 1 ? 0 : std::min(c->adj_fuse, smax));
            const int every = sadj > 0 ? kAdjGroup : 1;
            const int64_t top = a0 + (a1 - 1 - a0) / every * every;
            const int64_t nl = (top - a0 + kMaxFuse - 1) / kMaxFuse;           // launches
            int kind = fused_kind(d, every == 1 ? kRebuildKind : 0,
                                  nl > 0 ? (int)std::max<int64_t>(2, (top - a0 + nl - 1) / nl) : 2,
                                  true);
            if (!fused_shape(d, std::max(every, 2), kind).ok) kind = 0;
            for (int64_t n = a0; n < top;) {
                int s = 1;
                if (kind) {
                    s = launch_steps(d, kind, kMaxFuse, top - n);
                    s = s < every ? every : s / every * every;
                }
                at_status st = launch_1d(c, c->seg + (n - a0) * N, c->seg + (n + s - a0) * N, n, s,
                                         0, kind, s > 1 ? c->seg + (n - a0) * N : nullptr, every);
                if (st) return st;
                n += s;
            }
            // reverse launches over whole groups of levels, from the top (the
            // segment's last group may be short): as few as sadj allows, of even length
            for (int64_t nt = a1; sadj > 0 && nt > a0;) {
                const int64_t groups = (nt - a0 + kAdjGroup - 1) / kAdjGroup;
                const int64_t most = std::max(1, sadj / kAdjGroup);     // groups of a launch
                const int64_t left = (groups + most - 1) / most;            // launches
                const int64_t take = (groups + left - 1) / left;            // groups of this one
                const int s = (int)(nt - a0 - (groups - take) * kAdjGroup);
                AdjF f;
                f.lam_in = lcur;
                f.lam_out = loth;
                f.seg = c->seg;
                f.ring = c->ring;
                f.mu = c->mu;
                f.delays = c->delays;
                f.gnu = c->gnu;
                f.N = N;
                f.P = d.P;
                f.W = d.W;
                f.nt = nt;
                f.seg_n0 = a0;
                f.nsteps_total = nend;
                f.S = s;
                f.Rmu = c->lay.Rmu;
                f.L = c->cfg.L;
                f.stale = c->cfg.halo_mode;
                f.tpt = rg.tpt;
                f.nf = rg.nf;
                f.CT = rg.CT;
                f.RT = rg.RT;
                f.NT = rg.NT;
                f.coef = Step1D{};
                f.coef.nu = c->cfg.nu;
                f.coef.dt = c->cfg.dt;
                f.coef.c1 = d.c1[0];
                f.coef.c2 = d.c2[0];
                f.coef.cadv = c->cfg.adv_speed;
                f.coef.A1 = f.coef.dt * f.coef.c1;
                f.coef.A2 = f.coef.dt * (f.coef.nu * f.coef.c2);
                AT_HIP(launch_adj1d_fused(f, d.order, c->cfg.adv_mode == 1, c->cfg.arith == 1,
                                          rg.ppt, rg.nblocks,
                                          adj1d_fused_lds_bytes(d.order, s, rg.NT, c->cfg.L),
                                          c->st));
                std::swap(lcur, loth);
                nt -= s;
            }
            for (int64_t n = a1 - 1; sadj == 0 && n >= a0; --n) {
                Adj1D a;
                a.lam_in = lcur;
                a.lam_out = loth;
                a.u = c->seg + (n - a0) * N;
                a.ring = c->ring;
                a.mu = c->mu;
                a.delays = c->delays;
                a.gnu = c->gnu;
                a.N = N;
                a.P = d.P;
                a.W = d.W;
                a.n = n;
                a.nsteps_total = nend;
                a.R = c->lay.R;
                a.Rmu = c->lay.Rmu;
                a.L = c->cfg.L;
                a.stale = c->cfg.halo_mode;
                a.mslot0 = (int32_t)(n % a.Rmu);
                a.pad0 = 0;
                a.nu = c->cfg.nu;
                a.dt = c->cfg.dt;
                a.c1 = d.c1[0];
                a.c2 = d.c2[0];
                a.cadv = c->cfg.adv_speed;
                AT_HIP(launch_adj1d(a, d.order, c->cfg.adv_mode == 1, adj_blocks(d), c->st));
                std::swap(lcur, loth);
            }
        }
    }
    AT_HIP(launch_copy(grad_u0, lcur, N, c->st));
    AT_HIP(launch_gnu_final(c->gnu, c->lay.ngnu, grad_nu_dev, c->st));
    return AT_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Batched form: independent 1D instances advanced by shared launches
// ---------------------------------------------------------------------------

// Region kind (points per thread) and steps per launch of a batch's runs of up to
// `want` steps at a time (batch_plan); want 0: none yet
struct BatchPlan {
    int want = 0, kind = 16, steps = 1;
};

struct at_batch {
    int count = 0, order = 2;
    bool linear = false, fma = false;
    hipStream_t st = nullptr;
    std::vector<at_config> cfg;
    std::vector<Derived> d;
    std::vector<int> R;
    std::vector<int8_t *> delays;
    std::vector<double *> ring;
    double *ring_all = nullptr;      // the rings are one stretch of the workspace
    int64_t ring_all_doubles = 0;
    int64_t nsteps_max = 0;   // smallest over the instances
    int max_fuse = 1, fuse = 1;
    int variant = 0;          // 0 and 1: 16 points per thread or 32 (batch_plan), 2: 8, 3: 4
    BatchPlan plan;           // of the last run's steps
    int mf_ppt[3] = {1, 1, 1};   // steps-per-launch limit for 16, 8, 4 points per thread
    int64_t n = 0;
    // device tables (two slots: the run's s and its tail)
    Step1D *desc_dev[2] = {nullptr, nullptr};
    int2 *tbl_dev[2] = {nullptr, nullptr};
    int64_t tbl_cap = 0;
    int slot_s[2] = {0, 0};
    int64_t slot_blocks[2] = {0, 0};
    size_t slot_lds[2] = {0, 0};
    uint64_t slot_key[2] = {0, 0};
    std::vector<Step1D> hdesc[2];
    std::vector<int2> htbl[2];
    // cached graph of one whole run, captured on a private stream (the
    // caller's stream may be the null stream, which cannot be captured)
    hipStream_t cap = nullptr;
    bool has_graph = false;
    hipGraphExec_t gexec = nullptr;
    int64_t g_n0 = -1, g_nsteps = -1;
    int g_fuse = 0, g_variant = -1;
    uint64_t g_key = 0;
};

namespace {

uint64_t ptr_key(double *const *u, double *const *s, int count)
{
    uint64_t h = 1469598103934665603ULL;
    for (int j = 0; j < count; ++j) {
        h = (h ^ (uint64_t)(uintptr_t)u[j]) * 1099511628211ULL;
        h = (h ^ (uint64_t)(uintptr_t)s[j]) * 1099511628211ULL;
    }
    return h;
}

void drop_graph(at_batch *b)
{
    if (b->has_graph) (void)hipGraphExecDestroy(b->gexec);
    b->has_graph = false;
    b->gexec = nullptr;
}

// Whether launches of s steps take 32 points per thread instead of 16: half as many
// waves of 1.9 times the time a step, but rims half as large a part of a region, so
// where the batch fills the SIMDs many times over.  By the waves of the busiest SIMD
// and their time per step (fused_cost), and for 32 points what a wave whose lanes
// are tile faces takes longer.  Measured (us per step, 16 and 32 points): tiles of
// 256, order 4, 2^24 points: 16 steps 11.3 and 11.6, 32: 11.2 and 10.2, 48: 11.5 and
// 9.9; 2^22 points, 48: 3.07 and 3.41; tiles of 64, 2^24 points, 16: 14.7 and 17.5.
bool batch_takes_32(const at_batch *b, int s)
{
    double nb16 = 0.0, nb32 = 0.0, faces = 0.0;
    for (const Derived &d : b->d) {
        const FusedShape x = fused_shape(d, s, 16), y = fused_shape(d, s, 32);
        if (d.W % 32 != 0 || !x.ok || !y.ok) return false;
        nb16 += (double)x.nblocks;
        nb32 += (double)y.nblocks;
        faces += (double)y.nblocks * (1.03 + 6.0 * d.h / (double)d.W);
    }
    return std::ceil(nb32 / 1024.0) * (0.035 + 0.0205 * 32) * (faces / nb32) <
           std::ceil(nb16 / 1024.0) * (0.035 + 0.0205 * 16);
}

// Region kind and steps per launch of runs of nsteps steps: the variant's points per
// thread, or fewer where an instance's tiles do not take them (4 always fits: the
// tile widths are multiples of 16), and the number of steps set, as far as every
// instance's regions allow
BatchPlan batch_plan(const at_batch *b, int64_t nsteps)
{
    BatchPlan r;
    r.want = (int)std::min<int64_t>(b->fuse, nsteps);
    if (b->plan.want == r.want) return b->plan;
    r.kind = 4;
    for (int p = b->variant <= 1 ? 16 : variant_points(b->variant); p > 4; p /= 2) {
        bool ok = true;
        for (const Derived &d : b->d) ok = ok && d.W % p == 0 && fused_shape(d, 1, p).ok;
        if (ok) { r.kind = p; break; }
    }
    if (r.kind == 16 && batch_takes_32(b, r.want)) r.kind = 32;
    r.steps = r.want;
    for (const Derived &d : b->d)
        while (r.steps > 1 && !fused_shape(d, r.steps, r.kind).ok) --r.steps;
    return r;
}

at_status batch_tables(at_batch *b, int slot, int s, double *const *u, double *const *scr,
                       uint64_t key)
{
    const uint64_t k2 = key ^ ((uint64_t)s * 0x9E3779B97F4A7C15ULL) ^
                        ((uint64_t)b->plan.kind * 0xD1B54A32D192ED03ULL);
    if (b->slot_s[slot] == s && b->slot_key[slot] == k2) return AT_OK;
    drop_graph(b);    // a cached graph reads these tables
    std::vector<Step1D> &D = b->hdesc[slot];
    std::vector<int2> &T = b->htbl[slot];
    D.resize(b->count);
    T.clear();
    size_t lds = 0;
    for (int j = 0; j < b->count; ++j) {
        const Derived &d = b->d[j];
        const FusedShape ws = fused_shape(d, s, b->plan.kind);
        if (!ws.ok) return fail(AT_ERR_STATE, "batch: no region for %d steps per launch", s);
        Step1D &a = D[j];
        a.uin = u[j];
        a.uout = scr[j];
        a.ring = b->ring[j];
        a.delays = b->delays[j];
        a.N = d.N;
        a.P = d.P;
        a.W = d.W;
        a.n0 = 0;
        a.CH = 0;
        a.s = s;
        a.R = b->R[j];
        a.NT = ws.NT;
        a.tpt = ws.tpt;
        a.nf = ws.nf;
        a.CT = ws.CT;
        a.RT = ws.RT;
        a.stale = b->cfg[j].halo_mode;
        a.publish = 2;        // no edge tape: the last D levels of a launch
        a.RL = 0;
        a.slot0 = 0;          // set per launch by the batched kernel
        a.D = b->cfg[j].L + d.m - 1;
        a.levels = nullptr;
        a.nu = b->cfg[j].nu;
        a.dt = b->cfg[j].dt;
        a.c1 = d.c1[0];
        a.c2 = d.c2[0];
        a.cadv = b->cfg[j].adv_speed;
        a.A1 = a.dt * a.c1;
        a.A2 = a.dt * (a.nu * a.c2);
        for (int64_t c = 0; c < ws.nblocks; ++c) T.push_back(make_int2(j, (int)c));
        lds = std::max(lds, ws.lds);
    }
    if ((int64_t)T.size() > b->tbl_cap) return fail(AT_ERR_STATE, "batch block table overflow");
    AT_HIP(hipStreamSynchronize(b->st));
    AT_HIP(hipMemcpyAsync(b->desc_dev[slot], D.data(), D.size() * sizeof(Step1D),
                          hipMemcpyHostToDevice, b->st));
    AT_HIP(hipMemcpyAsync(b->tbl_dev[slot], T.data(), T.size() * sizeof(int2),
                          hipMemcpyHostToDevice, b->st));
    AT_HIP(hipStreamSynchronize(b->st));
    b->slot_s[slot] = s;
    b->slot_key[slot] = k2;
    b->slot_blocks[slot] = (int64_t)T.size();
    b->slot_lds[slot] = lds;
    return AT_OK;
}

// the launches of one run (recorded into a graph when capturing)
at_status batch_launches(at_batch *b, int64_t n0, int64_t nsteps, double *const *u,
                         double *const *scr, hipStream_t stream)
{
    int flip = 0;
    int64_t done = 0;
    // launches of even length (two lengths at most), an even number of them: a copy
    // back of every instance's field costs more than one (256 of them: 0.6 ms)
    while (done < nsteps) {
        const int64_t left = nsteps - done, n = launch_count(left, b->plan.steps, flip);
        const int s = (int)((left + n - 1) / n);
        const int slot = s == b->slot_s[0] ? 0 : 1;
        AT_HIP(launch_wave1d_batch(b->desc_dev[slot], b->tbl_dev[slot], b->slot_blocks[slot],
                                   b->order, b->linear, b->fma, b->plan.kind, n0 + done, flip,
                                   b->slot_lds[slot], stream));
        flip ^= 1;
        done += s;
    }
    if (flip)
        for (int j = 0; j < b->count; ++j)
            AT_HIP(launch_copy(u[j], scr[j], b->d[j].N, stream));
    return AT_OK;
}

}  // namespace

extern "C" {

static at_status batch_layout(const at_config *cfgs, int32_t count, std::vector<Derived> &ds,
                              std::vector<uint64_t> &off_delays, std::vector<uint64_t> &off_ring,
                              std::vector<int> &Rs, uint64_t &off_desc, uint64_t &off_tbl,
                              int64_t &tbl_cap, int &smax, int (&mf_ppt)[3], uint64_t &total)
{
    if (!cfgs || count < 1) return fail(AT_ERR_ARG, "batch needs at least one configuration");
    ds.resize(count);
    off_delays.resize(count);
    off_ring.resize(count);
    Rs.resize(count);
    smax = kMaxFuse;
    for (int j = 0; j < count; ++j) {
        at_status st = derive(&cfgs[j], ds[j]);
        if (st) return fail(st, "instance %d: %s", j, g_err.c_str());
        ds[j].fppt = step1d_points_per_thread();
        if (cfgs[j].dim != 1) return fail(AT_ERR_ARG, "instance %d: batched form is 1D", j);
        if (cfgs[j].record) return fail(AT_ERR_ARG, "instance %d: record mode not batched", j);
        if (cfgs[j].order != cfgs[0].order || cfgs[j].adv_mode != cfgs[0].adv_mode ||
            cfgs[j].arith != cfgs[0].arith)
            return fail(AT_ERR_ARG, "instance %d: all instances share order, adv_mode and arith", j);
        if (ds[j].W % step1d_points_per_thread() != 0)
            return fail(AT_ERR_SHAPE, "instance %d: tile width %lld is not a multiple of %d", j,
                        (long long)ds[j].W, step1d_points_per_thread());
        smax = std::min(smax, region_limit(ds[j]));
    }
    // steps-per-launch limit for each points-per-thread choice (16 gives the
    // largest regions, so the rings sized for it serve every choice)
    const int ppts[3] = {16, 8, 4};
    for (int i = 0; i < 3; ++i) {
        mf_ppt[i] = kMaxFuse;
        for (int j = 0; j < count; ++j) {
            Derived d = ds[j];
            d.fppt = ppts[i];
            mf_ppt[i] = std::min(mf_ppt[i], region_limit(d));
        }
        mf_ppt[i] = std::min(mf_ppt[i], smax);
    }
    uint64_t off = 0;
    tbl_cap = 0;
    for (int j = 0; j < count; ++j) {
        Rs[j] = cfgs[j].L + ds[j].m - 1 + smax;
        off_delays[j] = off;
        off = align_up(off + (uint64_t)cfgs[j].nsteps_max * (uint64_t)ds[j].F);
        int64_t most = 0;
        for (int p : {32, 16, 8, 4})
            for (int s = 1; s <= smax; ++s) most = std::max(most, fused_shape(ds[j], s, p).nblocks);
        tbl_cap += most;
    }
    for (int j = 0; j < count; ++j) {      // the rings together, cleared by one launch
        off_ring[j] = off;
        off = align_up(off + 8ull * (uint64_t)Rs[j] * (uint64_t)ds[j].P * 2 * ds[j].h);
    }
    off_desc = off;
    off = align_up(off + 2ull * count * sizeof(Step1D));
    off_tbl = off;
    off = align_up(off + 2ull * (uint64_t)tbl_cap * sizeof(int2));
    total = off;
    return AT_OK;
}

at_status at_batch_workspace_bytes(const at_config *cfgs, int32_t count, uint64_t *bytes)
{
    if (!bytes) return fail(AT_ERR_ARG, "null output");
    std::vector<Derived> ds;
    std::vector<uint64_t> od, orr;
    std::vector<int> Rs;
    uint64_t odesc, otbl, total;
    int64_t cap;
    int smax, mfp[3];
    at_status st = batch_layout(cfgs, count, ds, od, orr, Rs, odesc, otbl, cap, smax, mfp, total);
    if (st) return st;
    *bytes = total;
    return AT_OK;
}

at_status at_batch_init(const at_config *cfgs, int32_t count, void *workspace,
                        uint64_t workspace_bytes, at_batch **out)
{
    if (!out) return fail(AT_ERR_ARG, "null output");
    *out = nullptr;
    std::vector<Derived> ds;
    std::vector<uint64_t> od, orr;
    std::vector<int> Rs;
    uint64_t odesc, otbl, total;
    int64_t cap;
    int smax, mfp[3];
    at_status st = batch_layout(cfgs, count, ds, od, orr, Rs, odesc, otbl, cap, smax, mfp, total);
    if (st) return st;
    if (!workspace || ((uintptr_t)workspace) % kAlign)
        return fail(AT_ERR_ARG, "workspace NULL or not 256-byte aligned");
    if (workspace_bytes < total)
        return fail(AT_ERR_NOMEM, "workspace %llu bytes, need %llu",
                    (unsigned long long)workspace_bytes, (unsigned long long)total);
    for (int j = 0; j < count; ++j) {
        const at_config *c = &cfgs[j];
        if (c->delay_mode != AT_DELAY_HOST) continue;
        for (int64_t n = 0; n < c->nsteps_max; ++n) {
            const int64_t lim = std::min<int64_t>(c->L, std::max<int64_t>(0, n - ds[j].m + 1));
            for (int64_t f = 0; f < ds[j].F; ++f) {
                const int k = c->delays_host[n * ds[j].F + f];
                if (k < 0 || k > lim)
                    return fail(AT_ERR_DELAY, "instance %d: delay k[%lld][%lld] = %d outside 0..%lld",
                                j, (long long)n, (long long)f, k, (long long)lim);
            }
        }
    }
    at_batch *b = new (std::nothrow) at_batch;
    if (!b) return fail(AT_ERR_NOMEM, "host allocation failed");
    char *base = (char *)workspace;
    b->count = count;
    b->order = cfgs[0].order;
    b->linear = cfgs[0].adv_mode == 1;
    b->fma = cfgs[0].arith == 1;
    b->st = (hipStream_t)cfgs[0].stream;
    b->cfg.assign(cfgs, cfgs + count);
    b->d = ds;
    b->R = Rs;
    for (int i = 0; i < 3; ++i) b->mf_ppt[i] = mfp[i];
    b->max_fuse = mfp[0];
    b->fuse = cfgs[0].fuse_steps > 0 ? std::min<int>(cfgs[0].fuse_steps, b->max_fuse) : 1;
    b->nsteps_max = cfgs[0].nsteps_max;
    b->tbl_cap = cap;
    for (int s = 0; s < 2; ++s) {
        b->desc_dev[s] = (Step1D *)(base + odesc + (uint64_t)s * count * sizeof(Step1D));
        b->tbl_dev[s] = (int2 *)(base + otbl + (uint64_t)s * cap * sizeof(int2));
    }
    hipError_t e = hipSuccess;
    for (int j = 0; j < count && e == hipSuccess; ++j) {
        const at_config *c = &cfgs[j];
        b->cfg[j].delays_host = nullptr;
        b->nsteps_max = std::min<int64_t>(b->nsteps_max, c->nsteps_max);
        b->delays.push_back((int8_t *)(base + od[j]));
        b->ring.push_back((double *)(base + orr[j]));
        if (c->delay_mode == AT_DELAY_GENERATE)
            e = launch_delays(b->delays[j], c->nsteps_max, ds[j].F, c->L, ds[j].m, c->delay_dist,
                              c->delay_seed, b->st);
        else if (c->nsteps_max > 0)
            e = hipMemcpyAsync(b->delays[j], c->delays_host, (size_t)(c->nsteps_max * ds[j].F),
                               hipMemcpyHostToDevice, b->st);
    }
    // the rings follow each other (batch_layout), so one pass clears them all
    b->ring_all = (double *)(base + orr[0]);
    b->ring_all_doubles = (int64_t)((odesc - orr[0]) / 8);
    if (e == hipSuccess) e = launch_fill(b->ring_all, b->ring_all_doubles, 0.0, b->st);
    if (e == hipSuccess) e = hipStreamSynchronize(b->st);
    if (e != hipSuccess) {
        delete b;
        return fail(AT_ERR_HIP, "at_batch_init: %s", hipGetErrorString(e));
    }
    *out = b;
    return AT_OK;
}

void at_batch_free(at_batch *b)
{
    if (!b) return;
    drop_graph(b);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    delete b;
}

at_status at_batch_set_fuse(at_batch *b, int32_t s)
{
    if (!b) return fail(AT_ERR_ARG, "null batch");
    if (s < 1 || s > b->max_fuse)
        return fail(AT_ERR_ARG, "fuse_steps must be in 1..%d for this batch", b->max_fuse);
    b->fuse = s;
    b->plan = BatchPlan();
    return AT_OK;
}

at_status at_batch_set_variant(at_batch *b, int32_t v)
{
    if (!b) return fail(AT_ERR_ARG, "null batch");
    if (v < 0 || v > 3) return fail(AT_ERR_ARG, "batch variant must be in 0..3");
    const int idx = v <= 1 ? 0 : v - 1;               // 16, 8, 4 points per thread
    b->variant = v;
    b->plan = BatchPlan();
    b->max_fuse = b->mf_ppt[idx];
    b->fuse = std::min(b->fuse, b->max_fuse);
    b->slot_s[0] = b->slot_s[1] = 0;                  // tables are rebuilt for the new layout
    drop_graph(b);
    return AT_OK;
}

at_status at_batch_reset(at_batch *b)
{
    if (!b) return fail(AT_ERR_ARG, "null batch");
    AT_HIP(launch_fill(b->ring_all, b->ring_all_doubles, 0.0, b->st));
    b->n = 0;
    return AT_OK;
}

at_status at_batch_run(at_batch *b, double *const *u, double *const *scr, int64_t nsteps,
                       int32_t use_graph)
{
    if (!b || !u || !scr) return fail(AT_ERR_ARG, "null argument");
    if (nsteps < 0) return fail(AT_ERR_ARG, "nsteps < 0");
    if (b->n + nsteps > b->nsteps_max)
        return fail(AT_ERR_STATE, "batch run to step %lld beyond nsteps_max %lld",
                    (long long)(b->n + nsteps), (long long)b->nsteps_max);
    for (int j = 0; j < b->count; ++j)
        if (!u[j] || !scr[j] || u[j] == scr[j]) return fail(AT_ERR_ARG, "instance %d: bad fields", j);
    if (nsteps == 0) return AT_OK;
    const uint64_t key = ptr_key(u, scr, b->count);
    if (use_graph && b->has_graph && b->g_n0 == b->n && b->g_nsteps == nsteps &&
        b->g_fuse == b->fuse && b->g_variant == b->variant && b->g_key == key) {
        AT_HIP(hipGraphLaunch(b->gexec, b->st));
        b->n += nsteps;
        return AT_OK;
    }
    // the run's launches are s or s - 1 steps long (batch_launches)
    b->plan = batch_plan(b, nsteps);
    const int64_t nl = launch_count(nsteps, b->plan.steps, 0);
    const int s_long = (int)((nsteps + nl - 1) / nl);
    at_status st = batch_tables(b, 0, s_long, u, scr, key);
    if (st) return st;
    if (nsteps % nl != 0) {
        st = batch_tables(b, 1, s_long - 1, u, scr, key);
        if (st) return st;
    }
    if (!use_graph) {
        st = batch_launches(b, b->n, nsteps, u, scr, b->st);
        if (st) return st;
        b->n += nsteps;
        return AT_OK;
    }
    drop_graph(b);
    if (!b->cap) AT_HIP(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
    hipGraph_t g;
    AT_HIP(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
    st = batch_launches(b, b->n, nsteps, u, scr, b->cap);
    hipError_t e = hipStreamEndCapture(b->cap, &g);
    if (st) return st;
    if (e != hipSuccess) return fail(AT_ERR_HIP, "graph capture: %s", hipGetErrorString(e));
    e = hipGraphInstantiate(&b->gexec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) return fail(AT_ERR_HIP, "graph instantiate: %s", hipGetErrorString(e));
    b->has_graph = true;
    b->g_n0 = b->n;
    b->g_nsteps = nsteps;
    b->g_fuse = b->fuse;
    b->g_variant = b->variant;
    b->g_key = key;
    AT_HIP(hipGraphLaunch(b->gexec, b->st));
    b->n += nsteps;
    return AT_OK;
}

at_status at_batch_autotune(at_batch *b, double *const *u0, double *const *t1,
                            double *const *t2, int32_t trial_steps, int32_t *chosen)
{
    if (!b || !u0 || !t1 || !t2) return fail(AT_ERR_ARG, "null argument");
    if (b->n != 0) return fail(AT_ERR_STATE, "autotune needs a batch at step 0");
    if (trial_steps < 1 || trial_steps > b->nsteps_max)
        return fail(AT_ERR_ARG, "trial_steps must be in 1..nsteps_max");
    static const int cands[] = {1, 4, 8, 12, 16, 20, 24, 28, 32, 40, 48, 56, 64};
    hipEvent_t e0, e1;
    AT_HIP(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(AT_ERR_HIP, "at_batch_autotune: hipEventCreate failed");
    }
    // variant and steps per launch, the largest steps per launch first
    struct Trial { int variant, s; float ms; };
    std::vector<Trial> tr;
    at_status st = AT_OK;
    for (int v = 1; v <= 3 && st == AT_OK; ++v) {
        st = at_batch_set_variant(b, v);
        const int p = variant_points(v);
        bool ok = st == AT_OK;
        for (const Derived &d : b->d) ok = ok && d.W % p == 0 && fused_shape(d, 1, p).ok;
        if (!ok) continue;
        for (int ci = (int)(sizeof(cands) / sizeof(cands[0])) - 1; ci >= 0; --ci) {
            if (cands[ci] > b->max_fuse) continue;
            b->fuse = cands[ci];
            b->plan = BatchPlan();
            if (batch_plan(b, b->fuse).steps == b->fuse) tr.push_back({v, b->fuse, 1e30f});
        }
    }
    // every candidate twice in turn (the first run builds its tables), then those
    // within 10% of the best once more in the same way: an idle device's clock
    // takes some ten milliseconds to rise, at the first candidates' expense
    for (int round = 0; round < 2 && st == AT_OK; ++round) {
        float near = 1e30f;
        for (const Trial &t : tr) near = std::min(near, 1.1f * t.ms);
        for (size_t i = 0; i < tr.size() && st == AT_OK; ++i) {
            Trial &t = tr[i];
            if (round > 0 && t.ms > near) continue;
            st = at_batch_set_variant(b, t.variant);
            const int steps = trial_length(trial_steps, t.s, b->nsteps_max);
            for (int rep = 0; rep < 2 && st == AT_OK; ++rep) {
                st = at_batch_reset(b);
                hipError_t e = hipSuccess;
                for (int j = 0; j < b->count && st == AT_OK && e == hipSuccess; ++j)
                    e = launch_copy(t1[j], u0[j], b->d[j].N, b->st);
                b->fuse = t.s;
                b->plan = BatchPlan();
                if (st == AT_OK && e == hipSuccess) e = hipEventRecord(e0, b->st);
                if (st == AT_OK && e == hipSuccess) st = at_batch_run(b, t1, t2, steps, 0);
                if (st == AT_OK && e == hipSuccess) e = hipEventRecord(e1, b->st);
                if (st == AT_OK && e == hipSuccess) e = hipEventSynchronize(e1);
                float ms = 0.f;
                if (st == AT_OK && e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
                if (e != hipSuccess && st == AT_OK)
                    st = fail(AT_ERR_HIP, "at_batch_autotune: %s", hipGetErrorString(e));
                t.ms = std::min(t.ms, ms / (float)steps);
            }
        }
    }
    // a smaller count must be 2% faster to replace a larger one (fewer launches, and
    // fewer launch tails, on a near tie)
    size_t best = 0;
    for (size_t i = 1; i < tr.size(); ++i)
        if (tr[i].ms < tr[best].ms * 0.98f) best = i;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st) { b->n = 0; return st; }
    const int best_s = tr.empty() ? 1 : tr[best].s;
    st = at_batch_set_variant(b, tr.empty() ? 1 : tr[best].variant);
    if (st) return st;
    st = at_batch_reset(b);
    if (st) return st;
    AT_HIP(hipStreamSynchronize(b->st));
    b->fuse = best_s;
    b->plan = BatchPlan();
    if (chosen) *chosen = best_s;
    return AT_OK;
}

at_status at_batch_launch_shape(const at_batch *b, int64_t nsteps, int32_t *steps, int32_t *points)
{
    if (!b) return fail(AT_ERR_ARG, "null batch");
    if (nsteps < 1) return fail(AT_ERR_ARG, "nsteps < 1");
    const BatchPlan plan = batch_plan(b, nsteps);
    const int64_t nl = launch_count(nsteps, plan.steps, 0);
    if (steps) *steps = (int32_t)((nsteps + nl - 1) / nl);
    if (points) *points = plan.kind;
    return AT_OK;
}

at_status at_batch_query(const at_batch *b, int64_t *n, int32_t *fuse, int32_t *max_fuse,
                         int32_t *variant)
{
    if (!b) return fail(AT_ERR_ARG, "null batch");
    if (n) *n = b->n;
    if (fuse) *fuse = b->fuse;
    if (max_fuse) *max_fuse = b->max_fuse;
    if (variant) *variant = b->variant;
    return AT_OK;
}

}  // extern "C"
